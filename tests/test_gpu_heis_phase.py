"""Heisenberg sweeps in place, one launch per colour (no room for the second buffer; single sweeps; 3D L > 64), against
the oracle at the edges of the workgroups' shapes: rows of 1 .. 512 sites of a colour several to a workgroup
(more than a plane's in the smallest lattices), longer ones in segments, planes dealt out by fours."""
import math
import time

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
    spin.use_hip_allocator()
    yield
    spin.fault_alloc(-1)


def in_place(L, d, seed, replica=0):
    spin.fault_alloc(1)  # the spins' own buffer, then the second one
    h = spin.Heis(L, d, seed, replica)
    spin.fault_alloc(-1)
    return h


@pytest.mark.parametrize("L,d", [(4, 2), (6, 2), (34, 2), (100, 2), (130, 2), (258, 2), (340, 2), (510, 2), (514, 2), (1022, 2),
                                 (1026, 2), (2050, 2), (4, 3), (6, 3), (18, 3), (22, 3), (34, 3), (66, 3), (114, 3)])
def test_in_place_matches_oracle(oracle_mod, L, d):
    print("Heisenberg in place", L, d, flush=True)
    seed = workloads.seed(0x640 + L)
    h, ch = in_place(L, d, seed, 2), oracle_mod.HeisChain(L, d, seed, 2)
    for n, beta in [(1, 0.7), (2, 0.3), (1, math.inf), (1, 0.0), (3, 2.0)]:
        h.sweep(n, beta)
        ch.sweep(n, beta)
    assert np.array_equal(h.spins().reshape(-1, 4)[:, :3], np.asarray(ch.spins).reshape(L ** d, -1)[:, :3])
    h.close()


def test_planes_by_fours(oracle_mod):
    """3D L = 274: beyond 300 MB the XCDs go through the lattice together."""
    L, seed = 274, workloads.seed(0x641)
    print("Heisenberg in place", L, flush=True)
    h, ch = spin.Heis(L, 3, seed), oracle_mod.HeisChain(L, 3, seed, 0)
    h.sweep(1, 0.7)
    ch.sweep(1, 0.7)
    assert np.array_equal(h.spins().reshape(-1, 4)[:, :3], np.asarray(ch.spins).reshape(L ** 3, -1)[:, :3])
    h.close()


def test_rows_of_a_little_more_than_a_workgroup():
    """3D L = 520 costs about the 520^3 / 512^3 = 1.05 of L = 512 (with 256-site segments of a row it was 1.77: every
    other workgroup was nearly empty)."""
    us = {}
    for L in (512, 520):
        h = spin.Heis(L, 3, workloads.seed(0x642))
        best = math.inf
        for _ in range(4):
            h.synchronize()
            t0 = time.perf_counter()
            h.sweep(1, 0.7)
            h.synchronize()
            best = min(best, time.perf_counter() - t0)
        us[L] = best * 1e6
        h.close()
    assert us[520] <= 1.3 * us[512], us
