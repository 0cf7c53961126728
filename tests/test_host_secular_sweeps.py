"""How many sweeps the secular iteration takes, on the CPU: its mean on ordinary
problems and its slowest root on extreme ones.

Bounds: a model that matches f's slope alone takes 2.5 sweeps a root after the
first where the present one, with f's curvature, takes 1.7 to 2.2: at most 2.3.
The slowest of 16 million roots of the extreme kinds takes 18 sweeps: at most 24
here, and 32 eps of backward error as on ordinary problems."""
import os
import shutil
import subprocess

import pytest

HOST = os.path.join(os.path.dirname(os.path.abspath(__file__)), "host")


@pytest.fixture(scope="module")
def run(tmp_path_factory):
    if shutil.which("g++") is None:
        pytest.skip("g++ not available")
    at = tmp_path_factory.mktemp("sweeps")
    for name in ("secular_check", "secular_tail"):
        r = subprocess.run(["g++", "-std=gnu++17", "-O1", "-ffp-contract=off", "-Wno-unknown-pragmas", "-o",
                            str(at / name), os.path.join(HOST, name + ".cpp")], capture_output=True, text=True)
        assert r.returncode == 0, r.stderr[-4000:]

    def go(name, kind):
        r = subprocess.run([str(at / name), str(kind)], capture_output=True, text=True, timeout=120)
        assert r.returncode == 0, r.stderr[-2000:]
        return [float(x) for x in r.stdout.split()]

    return go


@pytest.mark.parametrize("kind", range(5), ids=["random", "jacobi", "graded", "clusters", "tiny weights"])
def test_mean_sweeps(run, kind):
    assert run("secular_check", kind)[3] <= 2.3


@pytest.mark.parametrize("kind", range(4), ids=["tiny weights", "graded", "clusters", "two weights"])
def test_slowest_root(run, kind):
    roots, capped, most, slow, worst = run("secular_tail", kind)
    assert roots > 30000 and capped == 0
    assert most <= 24 and slow <= 12, (most, slow)
    assert worst <= 32.0, worst
