"""Reverse mode with couplings far below the rest of the matrix, down to where
deflation decouples them (about 1e-15 of it): the derivative by such a coupling
is a difference that cancels, and deflated columns have their share in it.

Against the dense gradient (LAPACK eigenvectors), with weights smooth in the
eigenvalue, to the gradient gate of the other tests, 1e-7 of the largest weight;
equal weights give exactly 0 beside the diagonal."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

GATE = 1e-7


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


def _problem(g, n, p):
    """Random, the tears of the two topmost levels and an eighth of the couplings about 10^p."""
    d, e = g.uniform(-1.0, 1.0, n), g.uniform(-1.0, 1.0, n - 1)
    k = np.concatenate([g.choice(n - 1, min(n - 1, max(2, n // 8)), replace=False), [n // 2 - 1, max(n // 4 - 1, 0)]])
    e[k] = 10.0 ** p * g.choice([-1.0, 1.0], len(k)) * g.uniform(0.5, 2.0, len(k))
    return d, e


@pytest.mark.parametrize("n", [2, 3, 16, 100, 400, 700])
@pytest.mark.parametrize("leaf", [1, 4, 32])
def test_tiny_couplings(tde, n, leaf):
    g = np.random.default_rng(n + leaf)
    powers = [-300, -18, -16, -15, -14.5, -14, -13, -12, -11, -10, -9, -8, -4]
    for p in powers:
        print(f"[gpu-grad-tiny] n={n} leaf={leaf} couplings 1e{p}", flush=True)
        probs = [_problem(g, n, p) for _ in range(3)]
        d = np.concatenate([q[0] for q in probs])
        e = np.concatenate([np.append(q[1], 0.0) for q in probs])
        offs = [n * i for i in range(4)]
        lam, ckpt = tde.eigvals_ckpt(_t(d), _t(e), offs, leaf=leaf)
        w = np.cos(3.0 * lam.cpu().numpy())
        for wt in (w, np.ones_like(w)):
            gd, ge = (x.cpu().numpy() for x in tde.eigvals_backward(_t(d), _t(e), _t(wt), ckpt, offs, leaf=leaf))
            for b, (db, eb) in enumerate(probs):
                v, Q = np.linalg.eigh(np.diag(db) + np.diag(eb, 1) + np.diag(eb, -1))
                wb = wt[n * b:n * (b + 1)]
                ref_d, ref_e = (Q * Q) @ wb, 2.0 * (Q[:-1] * Q[1:]) @ wb
                top = np.abs(wb).max()
                assert np.abs(gd[n * b:n * (b + 1)] - ref_d).max() <= GATE * top, (p, b)
                assert np.abs(ge[n * b:n * (b + 1) - 1] - ref_e).max() <= GATE * top, (p, b)
