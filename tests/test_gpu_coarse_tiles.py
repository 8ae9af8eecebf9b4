"""Coarse-tile schedule where a workgroup holds several tiles and draws several hits ahead: numbers of
tiles that leave the last workgroup part filled, and hit counts around the four drawn at a time, against
the oracle.  Tolerance 0: spins, E and M are integers."""
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
    return torch


@pytest.mark.parametrize("model,d,L,T,k", [
    (0, 2, 48, 8, 4), (1, 2, 48, 8, 5), (0, 2, 80, 8, 9), (1, 2, 96, 16, 4), (0, 2, 32, 16, 9), (1, 2, 64, 32, 5),
    (0, 2, 128, 64, 9), (0, 3, 16, 8, 5), (1, 3, 48, 8, 4), (1, 3, 32, 16, 5),
])
def test_matches_oracle(oracle_mod, model, d, L, T, k):
    seed, cs = workloads.seed(0x48 + L + k), workloads.seed(0x12) if model else None
    print("coarse tiles", model, d, L, T, k, flush=True)
    lat = spin.Lattice(model, L, d, seed, coupling_seed=cs, replica=2)
    lat.set_schedule(spin.SPIN_SCHEDULE_COARSE, T, k)
    ch = oracle_mod.Chain(L, d, seed, 2, J=oracle_mod.couplings(L, d, cs, 0) if model else None)
    for beta in (0.45, 5.5, math.inf, 0.0):   # 5.5: one class accepts a single draw, the next none
        for got, want in zip(lat.sweep_record(1, beta, 1), ch.coarse_sweep(1, beta, T, k, every=1)):
            np.testing.assert_array_equal(got, want)
    np.testing.assert_array_equal(lat.spins(), ch.spins)
    lat.close()
