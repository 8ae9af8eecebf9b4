"""Pool calls of several size classes: one after another where they are short, else beside each other and beside larger
members, on streams that these leave free; the bits are those of the members alone, and a short call takes no
longer than a call for each class."""
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


def descs(model, L, d, count, first):
    return [dict(model=model, L=L, d=d, seed=workloads.seed(0x670), replica=first + r,
                 **({"coupling_seed": workloads.seed(0x14)} if model else {})) for r in range(count)]


def call_us(ds, n):
    b = spin.Batch(ds)
    best = math.inf
    for _ in range(6):
        b.sweep_device(n, 0.5, 0, None, None)
        b.synchronize()
        t0 = time.perf_counter()
        for _ in range(20):
            b.sweep_device(n, 0.5, 0, None, None)
        b.synchronize()
        best = min(best, (time.perf_counter() - t0) / 20)
    b.close()
    return best * 1e6


@pytest.mark.parametrize("count,n", [(4, 2), (400, 2), (4, 5)])
def test_short_call_of_two_classes(count, n):
    a, b = descs(1, 16, 3, count, 0), descs(0, 64, 2, count, 1000)
    both, apart = call_us(a + b, n), call_us(a, n) + call_us(b, n)
    assert both <= apart, (both, apart)


@pytest.mark.parametrize("bigs", [0, 1, 3, 5])
def test_members_are_the_lattices_alone(bigs):
    """Two short calls and a long one (side by side), with no, some and more larger members than there are streams."""
    ds = (descs(0, 512, 2, min(bigs, 3), 0) + descs(1, 72, 3, max(0, bigs - 3), 10) + descs(1, 16, 3, 5, 20) + descs(0, 64, 2, 5, 30) +
          descs(0, 32, 3, 3, 40) + descs(0, 256, 2, 2, 50))
    b = spin.Batch(ds)
    lats = [spin.Lattice(x["model"], x["L"], x["d"], x["seed"], coupling_seed=x.get("coupling_seed"), replica=x["replica"]) for x in ds]
    for n, beta, every in [(1, 0.5, 1), (2, 0.4, 0), (30, 0.6, 15)]:
        print("pool beside: bigs=%d n=%d" % (bigs, n), flush=True)
        rec = b.sweep(n, beta, every)
        for i, lat in enumerate(lats):
            if every:
                E, M = lat.sweep_record(n, beta, every)
                np.testing.assert_array_equal(rec[i][0], E)
                np.testing.assert_array_equal(rec[i][1], M)
            else:
                lat.sweep(n, beta)
    for i, lat in enumerate(lats):
        np.testing.assert_array_equal(b.spins(i), lat.spins())
        lat.close()
    b.close()
