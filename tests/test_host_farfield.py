"""The far-field series on the CPU against quadruple precision.

Bounds, of the sum of the terms' sizes: what the dropped terms leave (tde_far.h:
value 1.4e-17, derivatives 1.5e-14 and 7e-12, norm 5.0e-16, logarithm 2.3e-17)
plus rounding.  A moment is rounded at most ten times before it is added (the
reciprocal, u, its powers, the products), the sums of 50 poles add at most 7 eps
of the moments' sizes on average and Horner's rule two per term, with terms that
fall off like 4^-k; the sizes of the terms exceed the sum's by at most 5/3: under
32 half-eps = 16 eps.  The derivatives weight the k-th moment by k and k^2 / 2
and have limits twice and four times as wide.  Five terms fewer than 28 (or four
fewer than 16, two than 8) would leave 1e-14 or more."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
EPS = 2.0 ** -52


@pytest.mark.parametrize("contract", ["off", "fast"])
def test_series(tmp_path, contract):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    exe = str(tmp_path / "far_series")
    r = subprocess.run(["g++", "-std=gnu++17", "-O1", f"-ffp-contract={contract}", "-Wno-unknown-pragmas", "-o", exe,
                        os.path.join(ROOT, "tests", "host", "far_series.cpp")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0, r.stderr[-2000:]
    value, d1, d2, norm, log = (float(x) for x in r.stdout.split())
    assert value <= 1.4e-17 + 16 * EPS, value
    assert d1 <= 1.5e-14 + 32 * EPS, d1
    assert d2 <= 7e-12 + 64 * EPS, d2
    assert norm <= 5.0e-16 + 16 * EPS, norm
    assert log <= 2.3e-17 + 16 * EPS, log
