"""Up to four hits per tile load in 3D run without the table that later hits take their bounds from: either side of that
line against the oracle."""
import math

import numpy as np
import pytest

from paper_1006_3865_amd import spin, workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module", autouse=True)
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    spin.load()


@pytest.mark.parametrize("model,T,k", [(0, 8, 4), (0, 8, 5), (1, 8, 4), (1, 8, 5), (0, 16, 4), (0, 16, 5), (1, 16, 4), (1, 16, 5)])
def test_either_side(oracle_mod, model, T, k):
    seed, cs = workloads.seed(0x680 + k), workloads.seed(0x13) if model else None
    lat = spin.Lattice(model, 32, 3, seed, coupling_seed=cs, replica=1)
    lat.set_schedule(spin.SPIN_SCHEDULE_COARSE, T, k)
    ch = oracle_mod.Chain(32, 3, seed, 1, J=oracle_mod.couplings(32, 3, cs, 0) if model else None)
    for beta in (0.3, 1.9, 5.45, math.inf):
        print("coarse few hits", model, T, k, beta, flush=True)
        for got, want in zip(lat.sweep_record(1, beta, 1), ch.coarse_sweep(1, beta, T, k, every=1)):
            np.testing.assert_array_equal(got, want)
        np.testing.assert_array_equal(lat.spins(), ch.spins)
    lat.close()
