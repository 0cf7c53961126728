"""Reverse mode where a node inside the tree has a root exactly at a deflated
column's pole: small integer matrices with zero couplings, whose eigenvalues as
a whole may all be simple.

Against the dense gradient (LAPACK eigenvectors) where the spectrum is simple,
and for equal weights, whose gradient is 1 on the diagonal and 0 beside it, on
all of them.  The pass loses about eps / gap per level (three levels here, gaps
of the nodes over 0.05 or exactly 0): 1e-12."""
import itertools

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


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


@pytest.mark.parametrize("n,leaf", [(4, 1), (5, 1), (5, 2), (6, 2)])
def test_integer_matrices(tde, n, leaf):
    probs = [(d, e) for d in itertools.product([0.0, 1.0], repeat=n)
             for e in itertools.product([0.0, 1.0], repeat=n - 1)]
    print(f"[gpu-grad-equal] n={n} leaf={leaf} problems={len(probs)}", flush=True)
    d = np.array([p[0] for p in probs])
    e = np.array([p[1] + (0.0,) for p in probs])
    offs = [n * i for i in range(len(probs) + 1)]
    dv, ev = _t(d.ravel()), _t(e.ravel())
    lam, ckpt = tde.eigvals_ckpt(dv, ev, offs, leaf=leaf)
    w = np.tile(np.arange(1.0, n + 1), (len(probs), 1))
    for wt in (np.ones_like(w), w):
        gd, ge = (x.cpu().numpy().reshape(len(probs), n)
                  for x in tde.eigvals_backward(dv, ev, _t(wt.ravel()), ckpt, offs, leaf=leaf))
        for b in range(len(probs)):
            if wt is w:
                T = np.diag(d[b]) + np.diag(e[b, :-1], 1) + np.diag(e[b, :-1], -1)
                v, Q = np.linalg.eigh(T)
                if np.diff(v).min() < 1e-3:
                    continue
                ref_d, ref_e = (Q * Q) @ w[b], 2.0 * (Q[:-1] * Q[1:]) @ w[b]
            else:
                ref_d, ref_e = np.ones(n), np.zeros(n - 1)
            assert np.abs(gd[b] - ref_d).max() <= 1e-12, (probs[b], gd[b], ref_d)
            assert np.abs(ge[b, :-1] - ref_e).max() <= 1e-12, (probs[b], ge[b], ref_e)
