"""The host side of a requested-rows call on the CPU: tests/host/selrows_check.cpp
builds tde_api.cpp and tde_planner.cpp with g++ (address and undefined-behaviour
sanitizers) over a HIP runtime on host memory and fails every allocation,
copy and launch of a call in turn."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HOST = os.path.join(ROOT, "tests", "host")
CSRC = os.path.join(ROOT, "paper_2605_26599_amd", "csrc")


def test_selrows_host(tmp_path):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "selrows_check")
    cmd = ["g++", "-std=c++17", "-O1", "-g", "-fsanitize=address,undefined", "-fno-sanitize-recover=all",
           "-Wno-unknown-pragmas", "-DTDE_DEV=inline", "-I", os.path.join(HOST, "fake_hip"), "-o", exe,
           os.path.join(HOST, "selrows_check.cpp"), os.path.join(CSRC, "tde_api.cpp"),
           os.path.join(CSRC, "tde_planner.cpp")]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "selrows ok" in r.stdout, r.stdout[-2000:] + r.stderr[-4000:]
