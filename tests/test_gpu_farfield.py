"""Wide merges whose far poles enter through moment expansions, against the
oracle: spectra that keep every root (Jacobi recurrence matrices), at sizes
around a 64-root block's edges and the fewest far poles an expansion takes,
also with a gap inside a block, shifted into a narrow interval, and short.

Tolerance on eigenvalues: every level may deflate up to 8 eps max(|D|, 1) of
the scaled problem, at most 24 eps ||T||_1, and these trees have at most nine
levels: 256 eps ||T||_1.  Rows as everywhere: 1e-10 + 64 eps ||T|| / gap_k.
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


def _legendre(n):
    k = np.arange(1, n, dtype=np.float64)
    return np.zeros(n), k / np.sqrt(4.0 * k * k - 1.0)


def _matrix(kind, n):
    d, e = _legendre(n)
    if kind == "gap":  # two copies of [-1, 1], far apart and weakly coupled
        h = n // 3
        d2, e2 = _legendre(n - h)
        d, e = np.concatenate([d[:h], d2 + 9.0]), np.concatenate([e[:h - 1], [1e-3], e2])
    elif kind == "narrow":  # the whole spectrum within 2e-6 of 1
        d, e = 1.0 + 1e-6 * d, 1e-6 * e
    elif kind == "graded":  # widths over several orders of magnitude
        s = 10.0 ** (-4.0 * np.arange(n) / n)
        d, e = s * 2.0, -s[1:] * 0.9
    return d, e


@pytest.mark.parametrize("kind", ["plain", "gap", "narrow", "graded"])
@pytest.mark.parametrize("n", [513, 576, 577, 640, 703, 1025, 2111])
@pytest.mark.parametrize("wide_blocks", [None, 2])
def test_far_field_spectrum(tde, kind, n, wide_blocks):
    d, e = _matrix(kind, n)
    tol = 256.0 * EPS * tdgen.tnorm1(d, e)
    ref = oracle.eigvals(d, e)
    # wide blocks alone (eight waves), and beside regular tiles (four waves)
    for wide_min, fuse_few in [(2, 2), (600, 64)]:
        print(f"[gpu-far] {kind} n={n} wide_min={wide_min} blocks={wide_blocks}", flush=True)
        lam = tde.eigvals(_t(d), _t(e), wide_min=wide_min, fuse_few=fuse_few, wide_blocks=wide_blocks).cpu().numpy()
        assert np.all(np.diff(lam) >= 0.0)
        assert np.abs(lam - ref).max() <= tol, (n, np.abs(lam - ref).max() / tol)


@pytest.mark.parametrize("n", [577, 640, 1025, 2111])
def test_far_field_rows(tde, n):
    d, e = _matrix("plain", n)
    lr, r0, r1 = oracle.boundary_rows(d, e)
    gap = np.minimum(np.append(np.diff(lr), np.inf), np.insert(np.diff(lr), 0, np.inf))
    tol = 1e-10 + 64.0 * EPS * tdgen.tnorm1(d, e) / gap
    for wide_min, fuse_few in [(2, 2), (600, 64)]:
        tde.set_defaults(wide_min=wide_min, fuse_few=fuse_few)
        try:
            print(f"[gpu-far] rows n={n} wide_min={wide_min}", flush=True)
            lam, q0, q1 = (x.cpu().numpy() for x in tde.eigvals_rows(_t(d), _t(e)))
        finally:
            tde.set_defaults()
        assert np.abs(lam - lr).max() <= 256.0 * EPS * tdgen.tnorm1(d, e)
        assert np.all(np.abs(q0 - np.abs(r0)) <= tol)
        assert np.all(np.abs(q0 * q1 - r0 * r1) <= tol)


@pytest.mark.parametrize("n", [9000, 20001])
def test_far_field_distant(tde, n):
    """Merges with poles beyond 128 half-widths of a block, whose moments stop
    at eight terms (half of a Toeplitz merge's columns stay active), against
    4 sin^2(k pi / (2 (n + 1))); ten levels: 240 eps ||T||_1."""
    d, e = np.full(n, 2.0), np.full(n - 1, -1.0)
    ref = 4.0 * np.sin(np.arange(1, n + 1) * np.pi / (2.0 * (n + 1))) ** 2
    for wide_min, fuse_few in [(2, 2), (600, 64)]:
        print(f"[gpu-far] distant n={n} wide_min={wide_min}", flush=True)
        lam = tde.eigvals(_t(d), _t(e), wide_min=wide_min, fuse_few=fuse_few).cpu().numpy()
        assert np.all(np.diff(lam) >= 0.0)
        assert np.abs(lam - ref).max() <= 256.0 * EPS * 4.0
