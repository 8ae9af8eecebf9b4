"""Heisenberg sweeps several to a launch (tiles with halos in LDS) against the oracle."""
import math

import numpy as np
import pytest

from paper_1006_3865_amd import spin, workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def oracle_mod():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    import oracle
    spin.load()
    return oracle


@pytest.mark.parametrize("L,d", [(4, 2), (6, 2), (10, 2), (36, 2), (66, 2), (130, 2), (264, 2), (520, 2), (1000, 2),
                                 (4, 3), (10, 3), (18, 3), (34, 3), (64, 3), (66, 3)])
def test_several_sweeps_per_launch(oracle_mod, L, d):
    """Calls of several sweeps (tiles with halos in LDS; 3D L > 64: one launch per colour) at the edges of
    the tiles and with launches cut by records: every component bit for bit, E and |M| within 1e-9 a site."""
    print("Heisenberg several sweeps", L, d, flush=True)
    seed = workloads.seed(0x70 + L)
    h, ch = spin.Heis(L, d, seed, replica=1), oracle_mod.HeisChain(L, d, seed, 1)
    for n, every, beta in [(5, 0, 0.7), (1, 1, 0.3), (7, 3, 2.0), (2, 1, math.inf), (9, 9, 0.0), (4, 2, 1.1)]:
        if every:
            E, M = h.sweep_record(n, beta, every)
            for r in range(n // every):
                ch.sweep(every, beta)
                e, m = ch.measure()
                assert abs(E[r] - e) <= 1e-9 * L ** d and abs(M[r] - np.linalg.norm(m)) <= 1e-9 * L ** d
            ch.sweep(n % every, beta)
        else:
            h.sweep(n, beta)
            ch.sweep(n, beta)
        got = h.spins().reshape(-1, 4)
        assert np.array_equal(got[:, :3], np.asarray(ch.spins).reshape(L ** d, -1)[:, :3])
        assert (got[:, 3] == 0).all()
    h.close()
