"""The secular iteration's stopping rules on the CPU, in quadruple precision.

Bound: the rules accept |f| <= 8 eps (1 + rho sum |terms|), or a model step
whose successor could not move the root, with model terms up to 4 times f's
rounded four times (16 eps); evaluating f itself rounds too (8 eps allowed):
32 eps in all.
"""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    out = str(tmp_path_factory.mktemp("secular") / "secular_check")
    r = subprocess.run(["g++", "-std=gnu++17", "-O1", "-ffp-contract=off", "-Wno-unknown-pragmas", "-o", out,
                        os.path.join(ROOT, "tests", "host", "secular_check.cpp")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    return out


@pytest.mark.parametrize("kind", range(5), ids=["random", "jacobi", "graded", "clusters", "tiny weights"])
def test_secular_backward_error(exe, kind):
    r = subprocess.run([exe, str(kind)], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr[-2000:]
    roots, capped, worst, sweeps = (float(x) for x in r.stdout.split())
    assert roots > 500 and capped == 0
    assert worst <= 32.0, worst
