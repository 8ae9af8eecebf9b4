"""Kernels' LDS limits are set once per device and from any thread: the helper under a thread sanitizer, and no launch
function with a flag of its own."""
import glob
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1006_3865_amd", "csrc")


def test_threads_and_devices(tmp_path):
    gxx = shutil.which("g++")
    if not gxx:
        pytest.skip("no g++")
    exe = str(tmp_path / "once")
    src = os.path.join(ROOT, "tests", "helpers", "once_per_device.cpp")
    subprocess.check_call([gxx, "-std=c++17", "-O1", "-g", "-fsanitize=thread", "-pthread", "-I", CSRC, src, "-o", exe])
    out = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert out.returncode == 0 and "WARNING" not in out.stderr, out.stdout + out.stderr


def test_every_limit_is_set_by_the_helper():
    for path in glob.glob(os.path.join(CSRC, "*")):
        text = open(path).read()
        if os.path.basename(path) != "spin_launch.h":
            assert "hipFuncSetAttribute" not in text, path
        assert "static bool attr" not in text, path
