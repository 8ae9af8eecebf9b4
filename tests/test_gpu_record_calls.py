"""spin_sweep_record's host records: a call on a stream under capture is refused with nothing changed, long calls
give the same records as short ones, and what a handle keeps of their device arrays is bounded."""
import sys

import numpy as np
import pytest

from paper_1006_3865_amd import spin, workloads

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch():
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    spin.load()
    spin.use_hip_allocator()
    return torch


@pytest.mark.parametrize("L", [64, 256])
def test_capture_is_refused_and_changes_nothing(torch, oracle_mod, L):
    print("record call under capture: L=%d" % L, flush=True)
    sys.stdout.flush()
    stream = torch.cuda.Stream()
    seed = workloads.seed(0x630)
    lat = spin.Lattice(0, L, 2, seed)
    lat.set_stream(stream.cuda_stream)
    ch = oracle_mod.Chain(L, 2, seed, 0)
    Ea, Ma = lat.sweep_record(4, 0.4, 1)  # the device arrays are there
    Eo, Mo = ch.sweep(4, 0.4, every=1)
    np.testing.assert_array_equal(Ea, Eo)
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with pytest.raises(spin.SpinError) as ei:
        with torch.cuda.graph(g, stream=stream):
            lat.sweep_record(4, 0.4, 1)
    assert ei.value.code == spin.SPIN_ESTATE
    torch.cuda.synchronize()
    assert lat.t == 4
    np.testing.assert_array_equal(lat.spins(), ch.spins)
    Ea, Ma = lat.sweep_record(3, 0.4, 1)
    Eo, Mo = ch.sweep(3, 0.4, every=1)
    np.testing.assert_array_equal(Ea, Eo)
    np.testing.assert_array_equal(Ma, Mo)
    lat.close()


@pytest.mark.parametrize("n", [512, 513, 2000])
def test_long_calls(torch, n):
    """Up to 512 records come in one copy, more in one for each array."""
    seed = workloads.seed(0x631)
    a, b = spin.Lattice(0, 16, 2, seed), spin.Lattice(0, 16, 2, seed)
    Ea, Ma = a.sweep_record(n, 0.4, 1)
    parts = [b.sweep_record(k, 0.4, 1) for k in [100] * (n // 100) + ([n % 100] if n % 100 else [])]
    np.testing.assert_array_equal(Ea, np.concatenate([p[0] for p in parts]))
    np.testing.assert_array_equal(Ma, np.concatenate([p[1] for p in parts]))
    np.testing.assert_array_equal(a.spins(), b.spins())
    a.close()
    b.close()


def test_kept_memory_is_bounded(torch):
    base = spin.live_allocations()
    lat = spin.Lattice(0, 16, 2, workloads.seed(0x632))
    none = spin.live_allocations()
    lat.sweep_record(1000, 0.4, 1)
    assert spin.live_allocations() == none + 1
    lat.sweep_record(70000, 0.4, 1)  # 1.1 MB: not kept
    assert spin.live_allocations() == none
    lat.sweep_record(10, 0.4, 1)
    lat.close()
    assert spin.live_allocations() == base
