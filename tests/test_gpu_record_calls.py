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
