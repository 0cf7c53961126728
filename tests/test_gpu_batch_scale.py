"""Every problem of a batch is scaled by its own largest entry: batches of small
problems, many of which share a workgroup and a wave of that pass.

The solver works on T / 2^k with 2^k above the problem's largest entry, so a
batch times a power of two has the same eigenvalues times that power, bit for
bit, also where each problem has a power of its own; and a problem's place in
the batch changes nothing."""
import numpy as np
import pytest

import oracle
import tdgen

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


def _solve(tde, probs, scale, **kw):
    d = np.concatenate([p[0] * s for p, s in zip(probs, scale)])
    e = np.concatenate([np.append(p[1], 0.0)[: len(p[0])] * s for p, s in zip(probs, scale)])
    offs = np.concatenate([[0], np.cumsum([len(p[0]) for p in probs])]).tolist()
    return tde.eigvals_batched(_t(d), _t(e), offs, **kw).cpu().numpy(), offs


# sizes at which a wave's 64 and a workgroup's 1024 entries hold several problems, and a mix with larger ones
@pytest.mark.parametrize("sizes", [[1], [2], [3], [16], [63], [64], [65], [100], [257], [7, 300, 1, 40, 2000, 12]],
                         ids=str)
def test_batch_scales_by_powers_of_two(tde, sizes):
    count = max(40, 6000 // sum(sizes)) * len(sizes)
    probs = [tdgen.tridiag("uniform", sizes[i % len(sizes)], inst=i) for i in range(count)]
    g = np.random.default_rng(3)
    print(f"[gpu-scale] sizes={sizes} count={count}", flush=True)
    base, offs = _solve(tde, probs, np.ones(count))
    powers = [np.full(count, 2.0 ** -100), np.full(count, 2.0 ** 100), 2.0 ** g.integers(-100, 101, count)]
    for sc in powers:
        got, _ = _solve(tde, probs, sc)
        assert np.array_equal(got, base * np.repeat(sc, np.diff(offs)))
    for b in range(0, count, max(1, count // 40)):
        d, e = probs[b]
        assert np.abs(base[offs[b]:offs[b + 1]] - oracle.eigvals(d, e)).max() <= 2e-11 * tdgen.tnorm1(d, e)


@pytest.mark.parametrize("fam,n", [("clustered", 70), ("wilkinson", 66)])
@pytest.mark.parametrize("leaf", [1, 4])
def test_place_in_batch_changes_nothing(tde, fam, n, leaf):
    p = tdgen.tridiag(fam, n)
    print(f"[gpu-scale] places {fam} n={n} leaf={leaf}", flush=True)
    got, _ = _solve(tde, [p] * 2200, np.ones(2200), leaf=leaf)
    one = tde.eigvals(_t(p[0]), _t(p[1]), leaf=leaf).cpu().numpy()
    assert np.array_equal(got.reshape(2200, n), np.tile(one, (2200, 1)))


def test_gradients_of_small_scaled_problems(tde):
    """The reverse pass reads the same scales: dlambda/dT does not change when T
    is multiplied by a power of two."""
    count, n = 400, 24
    g = np.random.default_rng(4)
    d, e, w = (g.uniform(-1.0, 1.0, count * n) for _ in range(3))
    offs = [n * i for i in range(count + 1)]
    res = []
    for s in (1.0, 2.0 ** -100):
        print(f"[gpu-scale] gradients scale={s:g}", flush=True)
        lam, ckpt = tde.eigvals_ckpt(_t(d * s), _t(e * s), offs, leaf=8)
        gd, ge = tde.eigvals_backward(_t(d * s), _t(e * s), _t(w), ckpt, offs, leaf=8)
        res.append([x.cpu().numpy() for x in (lam / s, gd, ge)])
    for a, b in zip(*res):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("leaf", [1, 32])
def test_ends_of_the_range(tde, leaf):
    """Largest entries above 2^1023, and matrices of denormals: 64 of the
    smallest denormals of absolute error, or of eps of the norm."""
    n = 40
    d, e = tdgen.tridiag("wilkinson", n)
    ref = oracle.eigvals(d, e)
    big = 1.9 * 2.0 ** 1023 / np.abs(ref).max()
    for s, unit in ((2.0 ** -1072, 2.0 ** -1074), (2.0 ** -1030, 2.0 ** -1074), (big, 2.0 ** -52 * 1.9 * 2.0 ** 1023)):
        print(f"[gpu-scale] ends of the range scale={s:g} leaf={leaf}", flush=True)
        lam = tde.eigvals(_t(d * s), _t(e * s), leaf=leaf).cpu().numpy()
        assert np.isfinite(lam).all() and np.all(np.diff(lam) >= 0.0)
        assert np.abs(lam - ref * s).max() <= 64.0 * unit
