"""A pool's classes (dimension, model, workgroup size) run side by side: more classes than the pool has
further streams, calls back to back, members with nothing to do, and rows of odd and even numbers of words, each
lattice against the same lattice alone (whose chain is the oracle's).  Exact."""
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


def test_more_classes_than_streams():
    sizes = [(d, m, L) for d, edges in ((2, (8, 40, 64, 256, 400)), (3, (8, 16, 24, 48, 64))) for m in (0, 1) for L in edges]
    descs = [dict(model=m, L=L, d=d, seed=workloads.seed(0x900 + i), replica=i,
                  coupling_seed=workloads.seed(0x980) if m else 0, realisation=i % 2) for i, (d, m, L) in enumerate(sizes)]
    pool = spin.Batch(descs)
    lone = [spin.Lattice(c["model"], c["L"], c["d"], c["seed"], coupling_seed=c["coupling_seed"] if c["model"] else None,
                         realisation=c["realisation"], replica=c["replica"]) for c in descs]
    n = np.array([(3, 0, 5, 2)[i % 4] for i in range(len(descs))], dtype=np.int32)
    beta = np.array([(0.3, 0.9, float("inf"), 0.44)[i % 4 if i % 3 else 3] for i in range(len(descs))])
    for call in range(3):
        print("classes: call", call, flush=True)
        recs = pool.sweep(n, beta, 1)
        for i, lat in enumerate(lone):
            if n[i]:
                E, M = lat.sweep_record(int(n[i]), float(beta[i]), 1)
                np.testing.assert_array_equal(recs[i][0], E, err_msg=str(sizes[i]))
                np.testing.assert_array_equal(recs[i][1], M, err_msg=str(sizes[i]))
    for i, lat in enumerate(lone):
        np.testing.assert_array_equal(pool.spins(i), lat.spins(), err_msg=str(sizes[i]))
        lat.close()
    pool.close()
