"""Multi-spin-coded 3D lattices whose rows fill a part of a wavefront: the further lanes take other
strips of planes (as many as the strip height leaves), and sweeps march up and down in turn.  Every
number of parts, against the plane-streaming kernel; the chain is exact, so equality is."""
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


# (L, rows, planes): 256 has at most 2 parts, 128 at most 4; fewer where the strips do not divide L / parts
@pytest.mark.parametrize("L,rows,planes", [(256, 8, 2), (256, 4, 256), (128, 4, 2), (128, 8, 64), (128, 4, 4),
                                           (128, 8, 32)])
def test_parts_equal_streaming(L, rows, planes):
    cs, seed = workloads.seed(0x66), workloads.seed(0x67)
    a, b = spin.Msc(L, 3, cs, 2, seed, 9), spin.Msc(L, 3, cs, 2, seed, 9)
    a.set_kernel(2, rows, planes)
    b.set_kernel(1, 8, 16, 512 if L >= 256 else 256)
    print("parts", L, rows, planes, flush=True)
    for beta, n in ((0.9, 1), (1.6, 2), (float("inf"), 1)):   # odd counts: the march begins either way
        for x, y in zip(a.sweep_record(n, beta, 1), b.sweep_record(n, beta, 1)):
            np.testing.assert_array_equal(x, y)
    for system in (0, 31):
        np.testing.assert_array_equal(a.spins(system), b.spins(system))
    a.close()
    b.close()


# odd group counts and the smallest lattice; both sides of the size above which planes are streamed
@pytest.mark.parametrize("L,d", [(8, 2), (40, 2), (104, 2), (8, 3), (40, 3)])
def test_phase_kernel_matches_oracle(oracle_mod, L, d):
    cs, seed = workloads.seed(0x68), workloads.seed(0x69)
    m, ch = spin.Msc(L, d, cs, 4, seed, 3), oracle_mod.MscChain(L, d, cs, 4, seed, 3)
    print("phase", L, d, flush=True)
    assert m.kernel == 0
    for beta in (0.7, float("inf")):
        for x, y in zip(m.sweep_record(2, beta, 1), ch.sweep(2, beta, every=1)):
            np.testing.assert_array_equal(x, y)
    for system in (0, 31):
        np.testing.assert_array_equal(m.spins(system), ch.spins[system])
    m.close()


def test_streaming_beyond_the_cache():
    for L, d, kernel in ((2048, 2, 0), (4096, 2, 1), (200, 3, 0), (256, 3, 2)):
        m = spin.Msc(L, d, 1, 0, 1)
        assert m.kernel == kernel
        m.close()
