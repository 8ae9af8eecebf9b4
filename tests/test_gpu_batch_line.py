"""Where the classes of a pool call go side by side: calls on either side of the line, bit for bit and in time."""
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


def descs(model, L, d, count, first):
    return [dict(model=model, L=L, d=d, seed=workloads.seed(0x690), replica=first + r,
                 **({"coupling_seed": workloads.seed(0x14)} if model else {})) for r in range(count)]


def pool():
    return spin.Batch(descs(1, 16, 3, 4, 0) + descs(0, 64, 2, 4, 100))


def test_time_either_side():
    """Ten sweeps one class after another 45 us; twenty side by side 53 (one after another 68)."""
    b, best = pool(), {}
    for _ in range(8):
        for n in (10, 20):
            b.sweep_device(n, 0.5, 0, None, None)
            b.synchronize()
            t0 = time.perf_counter()
            for _ in range(30):
                b.sweep_device(n, 0.5, 0, None, None)
            b.synchronize()
            best[n] = min(best.get(n, math.inf), (time.perf_counter() - t0) / 30 * 1e6)
    b.close()
    assert best[20] <= 1.35 * best[10], best


@pytest.mark.parametrize("n", [18, 19])
def test_bits_either_side(n):
    """16^3 sites: 18 sweeps are estimated at 24.6 us, 19 at 25.9."""
    b = pool()
    lats = [spin.Lattice(x["model"], x["L"], x["d"], x["seed"], coupling_seed=x.get("coupling_seed"), replica=x["replica"])
            for x in descs(1, 16, 3, 4, 0) + descs(0, 64, 2, 4, 100)]
    b.sweep(n, 0.5, 0)
    for i, lat in enumerate(lats):
        lat.sweep(n, 0.5)
        np.testing.assert_array_equal(b.spins(i), lat.spins())
        lat.close()
    b.close()
