"""The kernels that AUTO's lattices name, run by name with their default tiles (AUTO itself runs most of these shapes
with several sweeps of a tile per launch), and the record calls and counts that only large lattices reach, against
the oracle or a count in numpy."""
import numpy as np
import pytest

from paper_1006_3865_amd import spin, workloads

pytestmark = pytest.mark.gpu

FUS, STR, RES = spin.SPIN_KERNEL_FUSED, spin.SPIN_KERNEL_STREAM, spin.SPIN_KERNEL_RESIDENT
CS = workloads.seed(0x11)


@pytest.fixture(scope="module", autouse=True)
def gpu():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    spin.load()
    spin.use_hip_allocator()


@pytest.mark.parametrize("kernel,model,L,d,tile", [
    (STR, 1, 1024, 2, (1024, 1, 8, 512)), (STR, 1, 128, 3, (128, 16, 4, 512)), (STR, 1, 72, 3, (72, 8, 4, 512)),
    (STR, 0, 72, 3, (72, 8, 4, 512)), (STR, 0, 160, 3, (160, 16, 4, 512)), (STR, 1, 200, 3, (200, 8, 4, 256)),
    (STR, 0, 320, 3, (320, 16, 8, 512)), (STR, 1, 384, 3, (384, 16, 8, 256)), (FUS, 0, 256, 3, (256, 16, 8, 576)),
    (FUS, 0, 640, 2, (128, 16, 0, 256)), (FUS, 0, 768, 2, (256, 32, 0, 256)), (FUS, 0, 1536, 2, (512, 16, 0, 256)),
    (FUS, 0, 400, 2, (16, 8, 0, 64)),
])
def test_default_tiles(oracle_mod, kernel, model, L, d, tile):
    print("default tile", kernel, model, L, d, flush=True)
    seed = workloads.seed(0x680 + L)
    lat = spin.Lattice(model, L, d, seed, coupling_seed=CS if model else None, replica=1)
    assert lat.kernel == kernel                        # the family that AUTO names ...
    lat.set_kernel(kernel)                             # ... by its own launches
    assert lat.tile == tile
    ch = oracle_mod.Chain(L, d, seed, 1, J=oracle_mod.couplings(L, d, CS, 0) if model else None)
    for n, beta, every in [(1, 0.3, 1), (2, 0.9, 2)]:
        E, M = lat.sweep_record(n, beta, every)
        Eo, Mo = ch.sweep(n, beta, every=every)
        np.testing.assert_array_equal(E, Eo)
        np.testing.assert_array_equal(M, Mo)
    np.testing.assert_array_equal(lat.spins(), ch.spins)
    lat.close()


def test_noalloc_records_beyond_the_scratch(oracle_mod):
    """2D L = 130: k_block's tiles of one row would need 130 pairs of counts a record, 3.1 MB for 1500 records; the
    allocation-free call has 2 MiB and takes the resident kernel, which needs none."""
    import torch
    L, n, seed = 130, 1500, workloads.seed(0x681)
    assert n * L * 16 > spin.NOALLOC_SCRATCH_BYTES
    lat = spin.Lattice(0, L, 2, seed)
    assert lat.kernel == RES
    E, M = (torch.zeros(n, dtype=torch.int64, device="cuda") for _ in range(2))
    lat.sweep_record_noalloc(n, 0.44, 1, E, M)
    ch = oracle_mod.Chain(L, 2, seed, 0)
    Eo, Mo = ch.sweep(n, 0.44, every=1)
    np.testing.assert_array_equal(E.cpu().numpy(), Eo)
    np.testing.assert_array_equal(M.cpu().numpy(), Mo)
    np.testing.assert_array_equal(lat.spins(), ch.spins)
    lat.close()


@pytest.mark.parametrize("L,d", [(264, 3), (5400, 2)])
def test_multi_spin_counts_over_several_chunks(oracle_mod, L, d):
    """E and M of lattices whose counting lanes take up their bit-sliced counters more than once (more than 64 sites
    a lane) and whose rows are several segments, the last one short, against sums over the spins in numpy."""
    print("multi-spin counts", L, d, flush=True)
    m = spin.Msc(L, d, CS, 3, workloads.seed(0x682))
    m.sweep(1, 0.8)
    E, M = m.measure()
    for s in (0, 13, 31):
        S = m.spins(s).reshape([L] * d)
        J = oracle_mod.couplings(L, d, CS, 3 + s).reshape([d] + [L] * d)
        e = 0
        for k in range(d):  # direction k is axis d - 1 - k
            e -= int(np.sum(S * np.roll(S, -1, d - 1 - k) * J[k], dtype=np.int64))
        assert (int(E[s]), int(M[s])) == (e, int(S.sum(dtype=np.int64)))
    m.close()


@pytest.mark.parametrize("replica", range(5))
def test_heisenberg_directions_of_many_draws(oracle_mod, replica):
    """Hot starts of 2D L = 4096: five of them draw 99.3 % of the 2^24 values of z = (w0 >> 8) 2^-23 - 1, whose root sqrt(1 - z z)
    has to be correctly rounded for the components to be the oracle's (which takes sqrtf)."""
    L, seed = 4096, workloads.seed(0x683)
    print("Heisenberg hot start", replica, flush=True)
    h = spin.Heis(L, 2, seed, replica)
    got = h.spins().reshape(-1, 4)[:, :3]
    h.close()
    assert np.array_equal(got, np.asarray(oracle_mod.HeisChain(L, 2, seed, replica).spins).reshape(L * L, -1)[:, :3])
