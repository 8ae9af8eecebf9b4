"""Lattices whose family works in place need one spin buffer: where the second one, for several sweeps of a tile
per launch, cannot be had, the constructor succeeds and every call gives the oracle's bits."""
import sys

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


def compare(lat, ch):
    for n, every in [(4, 2), (1, 1), (6, 0), (3, 1)]:
        if every:
            E, M = lat.sweep_record(n, 0.4, every)
            Eo, Mo = ch.sweep(n, 0.4, every=every)
            np.testing.assert_array_equal(E, Eo)
            np.testing.assert_array_equal(M, Mo)
        else:
            lat.sweep(n, 0.4)
            ch.sweep(n, 0.4)
        np.testing.assert_array_equal(lat.spins(), ch.spins)


@pytest.mark.parametrize("model,L,d,kernel", [(0, 96, 2, spin.SPIN_KERNEL_RESIDENT), (0, 96, 3, spin.SPIN_KERNEL_TILED),
                                              (0, 100, 3, spin.SPIN_KERNEL_GENERIC), (1, 50, 3, spin.SPIN_KERNEL_GENERIC)])
def test_no_room_for_a_second_buffer(oracle_mod, model, L, d, kernel):
    seed, cseed = workloads.seed(0x620 + L), workloads.seed(0x11) if model else None

    def make():
        return spin.Lattice(model, L, d, seed, coupling_seed=cseed)

    base = spin.live_allocations()
    whole = make()
    assert whole.kernel == kernel
    blocks = spin.live_allocations() - base
    whole.close()
    J = oracle_mod.couplings(L, d, cseed, 0) if model else None
    # the last allocation of the constructor is the second buffer
    print("second buffer: model=%d d=%d L=%d" % (model, d, L), flush=True)
    sys.stdout.flush()
    spin.fault_alloc(blocks - 1)
    lat = make()
    assert spin.live_allocations() - base == blocks - 1
    spin.fault_alloc(-1)
    compare(lat, oracle_mod.Chain(L, d, seed, 0, J=J))
    lat.close()
    assert spin.live_allocations() == base


def test_no_room_for_the_record_counts(oracle_mod):
    """k_block's counts of a record (a pair a tile) cannot be had, the family's own (none: one workgroup) need no room."""
    L, d, seed = 180, 2, workloads.seed(0x621)
    lat = spin.Lattice(0, L, d, seed)
    assert lat.kernel == spin.SPIN_KERNEL_RESIDENT
    ch = oracle_mod.Chain(L, d, seed, 0)
    import torch
    E, M = (torch.zeros(8, dtype=torch.int64, device="cuda") for _ in range(2))
    spin.fault_alloc(0)
    try:
        lat.sweep_record_device(8, 0.4, 1, E, M)
    finally:
        spin.fault_alloc(-1)
    Eo, Mo = ch.sweep(8, 0.4, every=1)
    np.testing.assert_array_equal(E.cpu().numpy(), Eo)
    np.testing.assert_array_equal(M.cpu().numpy(), Mo)
    np.testing.assert_array_equal(lat.spins(), ch.spins)
    lat.close()
