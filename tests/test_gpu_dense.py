"""Dense front end (tde_dense_eigvals) through the C-ABI: Householder
reduction of a dense symmetric matrix on the device, then the boundary-row
solve.

Parity: the eigenvalues of A against the oracle (textbook Householder
reduction plus bisection) at sizes it finishes in seconds; at larger sizes
against a prescribed spectrum (A = Q diag(lambda) Q^T with a seeded random
orthogonal Q), which fixes every eigenvalue exactly.  Gate: max |dlambda| <=
2e-11 ||A||_1, the tridiagonal path's gate with A's 1-norm.  The reduced
tridiagonal itself must keep trace and Frobenius norm.
"""
import ctypes

import numpy as np
import pytest

import oracle
import tdgen

pytestmark = pytest.mark.gpu

GATE = 2e-11


def _step(msg):
    print(f"[gpu-dense] {msg}", flush=True)


@pytest.fixture(scope="module")
def tde():
    import torch

    import paper_2605_26599_amd as m

    assert torch.cuda.is_available()
    m.lib()
    return m


def _sym(n, seed, kind):
    g = np.random.default_rng(seed)
    if kind == "random":
        B = g.uniform(-1.0, 1.0, (n, n))
        return 0.5 * (B + B.T), None
    Q, R = np.linalg.qr(g.standard_normal((n, n)))
    Q = Q * np.sign(np.diag(R))[None, :]
    if kind == "clustered":
        lam = np.sort(np.concatenate([np.full(n // 2, 0.5) + 1e-9 * g.standard_normal(n // 2),
                                      g.uniform(-1.0, 1.0, n - n // 2)]))
    else:
        lam = np.sort(g.uniform(-1.0, 1.0, n))
    A = Q @ np.diag(lam) @ Q.T
    return 0.5 * (A + A.T), lam


def _t(x):
    import torch

    return torch.from_numpy(np.ascontiguousarray(x, dtype=np.float64)).to("cuda:0")


def _norm1(A):
    return float(np.abs(A).sum(axis=0).max()) if A.size else 0.0


@pytest.mark.parametrize("kind", ["random", "prescribed", "clustered"])
def test_dense_matches_oracle(tde, kind):
    for n in [1, 2, 3, 5, 31, 32, 33, 34, 64, 65, 97, 200, 333]:
        A, _ = _sym(n, 100 + n, kind)
        _step(f"dense {kind} n={n}")
        lam, d, e = tde.dense_eigvals(_t(A), return_tridiagonal=True)
        lam, d, e = lam.cpu().numpy(), d.cpu().numpy(), e.cpu().numpy()
        ref = oracle.dense_eigvals(A)
        tol = GATE * max(_norm1(A), 1e-300)
        assert np.abs(lam - ref).max() <= tol, (n, float(np.abs(lam - ref).max()), tol)
        # the reduced tridiagonal: same spectrum, trace and Frobenius norm
        assert np.abs(oracle.eigvals(d, e) - ref).max() <= tol
        assert abs(d.sum() - np.trace(A)) <= 1e-12 * max(1.0, np.abs(A).sum())
        fro = float(np.sum(A * A))
        assert abs((d @ d + 2.0 * e @ e) - fro) <= 1e-12 * max(fro, 1.0)


@pytest.mark.parametrize("n", [1024, 4096])
def test_dense_prescribed_spectrum_large(tde, n):
    A, lam_exact = _sym(n, 7, "prescribed")
    _step(f"dense prescribed spectrum n={n}")
    lam = tde.dense_eigvals(_t(A)).cpu().numpy()
    err = float(np.abs(lam - lam_exact).max())
    print(f"dense n={n}: max|dlambda| = {err:.3e} = {err / _norm1(A):.3e} ||A||_1")
    assert err <= GATE * _norm1(A)
    lam2 = tde.dense_eigvals(_t(A)).cpu().numpy()
    assert np.array_equal(lam, lam2), "repeat differs"


def test_dense_leading_dimension_and_overwrite(tde):
    """A stored with lda > n (padding rows never read); overwrite=True gives
    the same eigenvalues as the copy; n = 0 is a no-op."""
    import torch

    n, lda = 150, 157
    A, _ = _sym(n, 3, "random")
    P = np.full((n, lda), np.nan)  # column-major with padding: column j = P[j, :]
    P[:, :n] = A  # symmetric, so row j of A is column j
    Pd = _t(P)
    lam = torch.empty(n, dtype=torch.float64, device="cuda:0")
    L = tde.lib()
    nb = L.tde_dense_workspace_bytes(n, None)
    ws = torch.empty(nb, dtype=torch.uint8, device="cuda:0")
    stream = torch.cuda.current_stream().cuda_stream
    rc = L.tde_dense_eigvals(Pd.data_ptr(), n, lda, lam.data_ptr(), None, None, ws.data_ptr(), nb, stream, None)
    assert rc == tde.TDE_OK
    assert L.tde_get_status(ws.data_ptr(), stream) == tde.TDE_OK
    ref = oracle.dense_eigvals(A)
    assert np.abs(lam.cpu().numpy() - ref).max() <= GATE * _norm1(A)
    assert np.isnan(Pd.cpu().numpy()[:, n:]).all()
    assert L.tde_dense_eigvals(Pd.data_ptr(), n, n - 1, lam.data_ptr(), None, None, ws.data_ptr(), nb, stream,
                               None) == tde.TDE_EINVAL
    assert L.tde_dense_eigvals(Pd.data_ptr(), n, lda, lam.data_ptr(), None, None, ws.data_ptr(), nb - 1, stream,
                               None) == tde.TDE_EINVAL
    B = _t(A)
    lam_ow = tde.dense_eigvals(B, overwrite=True).cpu().numpy()
    assert np.array_equal(lam_ow, tde.dense_eigvals(_t(A)).cpu().numpy())
    assert tde.dense_eigvals(torch.zeros((0, 0), dtype=torch.float64, device="cuda:0")).numel() == 0


@pytest.mark.parametrize("n", [63, 66, 127, 128, 129, 130, 193, 257, 321])
def test_dense_tile_edges(tde, n):
    """Sizes around the 64-row tiles and blocks of the reduction's kernels."""
    A, _ = _sym(n, 900 + n, "random")
    _step(f"dense tile edge n={n}")
    lam, d, e = (x.cpu().numpy() for x in tde.dense_eigvals(_t(A), return_tridiagonal=True))
    ref = oracle.dense_eigvals(A)
    tol = GATE * _norm1(A)
    assert np.abs(lam - ref).max() <= tol
    # an orthogonal reduction keeps the Frobenius norm
    fro = float(np.sum(A * A))
    assert abs((d @ d + 2.0 * e @ e) - fro) <= 1e-12 * fro


@pytest.mark.parametrize("n", [4097, 4200])
def test_dense_large_tiles(tde, n):
    """Above 4096 rows a tile has several subtiles; two reflections around a
    known spectrum fix every eigenvalue."""
    g = np.random.default_rng(n)
    lam = np.sort(g.uniform(-1.0, 1.0, n))
    A = np.diag(lam)
    for _ in range(2):
        u = g.standard_normal(n)
        u /= np.linalg.norm(u)
        w = A @ u
        A -= 2.0 * np.outer(u, w - (u @ w) * u) + 2.0 * np.outer(w - (u @ w) * u, u)
    A = 0.5 * (A + A.T)
    # H A H = A - 2 u w^T - 2 w u^T + 4 (u.w) u u^T, as applied above
    _step(f"dense large tiles n={n}")
    out = tde.dense_eigvals(_t(A)).cpu().numpy()
    assert np.abs(out - lam).max() <= GATE * _norm1(A)
    assert np.array_equal(out, tde.dense_eigvals(_t(A)).cpu().numpy()), "repeat differs"
