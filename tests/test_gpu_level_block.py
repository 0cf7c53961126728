"""Whole merges in one workgroup (every array in LDS, one thread per column):
merge sizes at the edges of the workgroup shapes, against the oracle, alone
and as a level of many merges (other workgroup shapes).

Tolerance: at most nine levels of up to 24 eps ||T||_1 of deflation each, as
for the wide merges: 256 eps ||T||_1.
"""
import numpy as np
import pytest

import oracle
import tdgen

pytestmark = pytest.mark.gpu

EPS = np.finfo(float).eps


@pytest.fixture(scope="module")
def tde():
    import torch

    import paper_2605_26599_amd as m

    assert torch.cuda.is_available()
    m.lib()
    return m


def _t(x):
    import torch

    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float64)).to("cuda:0")


@pytest.mark.parametrize("fam", ["uniform", "toeplitz", "clustered", "wilkinson"])
@pytest.mark.parametrize("n", [2, 3, 15, 16, 17, 33, 63, 64, 65, 127, 128, 129, 255, 256, 257, 511, 512, 513])
def test_level_block_edges(tde, fam, n):
    d, e = tdgen.tridiag(fam, n, cfg=tdgen.CFG_TEST)
    ref = oracle.eigvals(d, e)
    tol = 256.0 * EPS * tdgen.tnorm1(d, e)
    print(f"[gpu-level] {fam} n={n}", flush=True)
    lam = tde.eigvals(_t(d), _t(e if n > 1 else np.zeros(1)), leaf=1).cpu().numpy()
    assert np.abs(lam - ref).max() <= tol
    # the same problem many times over: levels of many merges
    B = 300 if n > 128 else 1100
    if n > 257:
        return
    D, E = np.tile(d, B), np.tile(np.append(e, 0.0), B)
    out = tde.eigvals_batched(_t(D), _t(E), [n * b for b in range(B + 1)], leaf=1).cpu().numpy().reshape(B, n)
    assert np.abs(out - ref).max() <= tol
