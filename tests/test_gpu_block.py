"""Several sweeps per launch (k_block; k_whole for the smallest lattices): AUTO handles whose calls of several sweeps run tiles with
halos in LDS, against the oracle bit for bit, at the edges of the tiles (narrow last tiles, rows of
one or a few groups, halos wider than the lattice), for rows of L % 8 != 0, and at the bounds where
the call falls back to single sweeps (n = 1 in place, a class with T = 1 beside one with T = 0)."""
import math
import sys

import numpy as np
import pytest

from paper_1006_3865_amd import spin, workloads

pytestmark = pytest.mark.gpu

CS = workloads.seed(0x11)


@pytest.fixture(scope="module")
def oracle_mod():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    import oracle
    spin.load()
    spin.use_hip_allocator()
    return oracle


def compare(oracle, model, L, d, sched, replica=3):
    seed = workloads.seed(0x500 + L)
    print("block: model=%d d=%d L=%d %r" % (model, d, L, sched), flush=True)
    sys.stdout.flush()
    lat = spin.Lattice(model, L, d, seed, coupling_seed=CS if model else None, replica=replica)
    ch = oracle.Chain(L, d, seed, replica, J=oracle.couplings(L, d, CS, 0) if model else None)
    for n, beta, every in sched:
        if every:
            E, M = lat.sweep_record(n, beta, every)
            Eo, Mo = ch.sweep(n, beta, every=every)
            np.testing.assert_array_equal(E, Eo)
            np.testing.assert_array_equal(M, Mo)
        else:
            lat.sweep(n, beta)
            ch.sweep(n, beta)
        np.testing.assert_array_equal(lat.spins(), ch.spins)
        assert lat.t == ch.t
        assert lat.measure() == ch.measure()
    lat.close()


SCHED = [(9, 0.44, 1), (1, 0.3, 1), (2, 0.5, 0), (8, 0.0, 3), (5, math.inf, 1), (7, 3.0, 2), (3, 0.4, 5)]


@pytest.mark.parametrize("model", [0, 1])
@pytest.mark.parametrize("L", [8, 16, 32, 40, 64, 72, 96, 136, 264, 520, 10, 12, 14, 34, 36, 38, 46, 62, 100, 250, 510])
def test_2d(oracle_mod, L, model):
    compare(oracle_mod, model, L, 2, SCHED + [(4, 5.45, 1)])


@pytest.mark.parametrize("model", [0, 1])
@pytest.mark.parametrize("L", [8, 16, 24, 32, 40, 72, 10, 12, 14, 18, 20, 22, 26, 50])
def test_3d(oracle_mod, L, model):
    compare(oracle_mod, model, L, 3, SCHED + [(4, 2.73, 1)])


@pytest.mark.parametrize("model,L,d,n", [(0, 1000, 2, 17), (0, 2056, 2, 8), (1, 1002, 2, 8), (0, 4104, 2, 4),
                                         (0, 100, 3, 10), (1, 128, 3, 6), (0, 200, 3, 4), (0, 256, 3, 4),
                                         (1, 250, 3, 2)])
def test_larger(oracle_mod, model, L, d, n):
    compare(oracle_mod, model, L, d, [(n, 0.44, 2), (n + 1, 0.7, 3)])


def test_switching_and_buffers(oracle_mod):
    """Calls that run k_block between calls on named families, a caller's spins and another start index."""
    L, d, seed = 96, 3, workloads.seed(0x560)
    lat = spin.Lattice(0, L, d, seed)
    ch = oracle_mod.Chain(L, d, seed)
    for kernel, n in [(spin.SPIN_KERNEL_AUTO, 3), (spin.SPIN_KERNEL_TILED, 2), (spin.SPIN_KERNEL_AUTO, 4),
                      (spin.SPIN_KERNEL_GENERIC, 1), (spin.SPIN_KERNEL_AUTO, 2)]:
        lat.set_kernel(kernel)
        E, M = lat.sweep_record(n, 0.3, 1)
        Eo, Mo = ch.sweep(n, 0.3, every=1)
        np.testing.assert_array_equal(E, Eo)
        np.testing.assert_array_equal(M, Mo)
    np.testing.assert_array_equal(lat.spins(), ch.spins)
    other = spin.Lattice(0, L, d, seed)
    other.set_spins(lat.spins())
    other.t = lat.t
    other.sweep(5, 0.3)
    lat.sweep(5, 0.3)
    np.testing.assert_array_equal(other.spins(), lat.spins())
    lat.close()
    other.close()


@pytest.mark.parametrize("L,d,n", [(96, 3, 4), (96, 3, 5), (100, 3, 4), (256, 2, 6), (48, 2, 3)])
def test_buffer_after_a_call(oracle_mod, L, d, n):
    """The current buffer after a call is the one the family's own launches would leave: in place, or
    swapped once per sweep."""
    lat = spin.Lattice(0, L, d, 5)
    pingpong = lat.kernel in (spin.SPIN_KERNEL_FUSED, spin.SPIN_KERNEL_STREAM)
    first = spin.spin_device_spins(lat.h)
    lat.sweep(n, 0.4)
    assert (spin.spin_device_spins(lat.h) == first) == (not pingpong or n % 2 == 0)
    lat.close()


def test_noalloc_beyond_scratch_still_runs(oracle_mod):
    """Records that fit the allocation-free call's scratch by the family's own partials stay accepted."""
    import torch
    L, n = 1000, 60
    per = spin.NOALLOC_SCRATCH_BYTES // 16 // n
    a, b = spin.Lattice(0, L, 2, 7), spin.Lattice(0, L, 2, 7)
    E, M = (torch.zeros(n, dtype=torch.int64, device="cuda") for _ in range(2))
    F, N = (torch.zeros(n, dtype=torch.int64, device="cuda") for _ in range(2))
    assert per > 0
    a.sweep_record_noalloc(n, 0.44, 1, E, M)
    b.sweep_record_device(n, 0.44, 1, F, N)
    torch.cuda.synchronize()
    assert torch.equal(E, F) and torch.equal(M, N)
    np.testing.assert_array_equal(a.spins(), b.spins())
    a.close()
    b.close()
