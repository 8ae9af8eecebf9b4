"""A tuning record from before the kernels of several sweeps per launch (no ninth field) keeps its family and tile and
does not keep a call of several sweeps from them; records with the field say which."""
import os
import subprocess
import sys

import pytest

from paper_1006_3865_amd import spin

pytestmark = pytest.mark.gpu

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CODE = r"""
import sys, time
sys.path.insert(0, %r)
import torch
from paper_1006_3865_amd import spin
spin.load()
lat = spin.Lattice(0, 1024, 2, 5)
print("family", lat.kernel, *lat.tile)
best = {}
for _ in range(5):
    for k in (0, spin.SPIN_KERNEL_FUSED):
        lat.set_kernel(k)
        lat.sweep(40, 0.44)
        lat.synchronize()
        t0 = time.perf_counter()
        for _ in range(5):
            lat.sweep(40, 0.44)
        lat.synchronize()
        best[k] = min(best.get(k, 1e9), time.perf_counter() - t0)
print("ratio", best[0] / best[spin.SPIN_KERNEL_FUSED])
""" % ROOT


@pytest.mark.parametrize("field,slow", [("", False), (" 1", False), (" 0", True)])
def test_record(tmp_path, field, slow):
    import torch
    if not torch.cuda.is_available():
        pytest.fail("no GPU visible")
    arch = torch.cuda.get_device_properties(0).gcnArchName.split(":")[0]
    path = str(tmp_path / "tune.txt")
    with open(path, "w") as f:
        f.write("lattice %s 0 1024 2 %d 256 32 0 256%s\n" % (arch, spin.SPIN_KERNEL_FUSED, field))
    out = subprocess.run([sys.executable, "-c", CODE], capture_output=True, text=True, timeout=120,
                         env=dict(os.environ, SPIN_TUNE_CACHE=path))
    assert out.returncode == 0, out.stderr
    lines = dict(ln.split(None, 1) for ln in out.stdout.splitlines() if " " in ln)
    assert lines["family"].split() == [str(spin.SPIN_KERNEL_FUSED), "256", "32", "0", "256"]
    # k_block takes about 0.3 of the family's time here
    assert (float(lines["ratio"]) > 0.8) == slow, out.stdout
