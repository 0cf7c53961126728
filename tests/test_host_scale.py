"""The scale of a problem on the CPU, from the smallest denormal to the largest
number (tests/host/scale_check.cpp)."""
import os
import shutil
import subprocess

import pytest

HOST = os.path.join(os.path.dirname(os.path.abspath(__file__)), "host")


def test_scale_range(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "scale_check")
    r = subprocess.run(["g++", "-std=gnu++17", "-O1", "-Wno-unknown-pragmas", "-o", exe,
                        os.path.join(HOST, "scale_check.cpp")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=60)
    assert r.returncode == 0 and "scale ok" in r.stdout, r.stdout
