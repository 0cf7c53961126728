"""The work that a user of this library has it do, as timed cases.

Every case is one pass through the Python entry points: single tridiagonals
(out of the box and with tuned launch options), batches, the reverse mode, the
dense front end, eigenvector rows and the splitting driver.  Inputs are seeded
synthetic matrices of the families the tests and the benchmark use, FP64 (the
only type the library takes), resident on the GPU before the pass.
"""
import math
import random

import numpy as np
import torch

import paper_2605_26599_amd as tde

NO_WIDE = 1 << 30  # "no wide sweeps" as the autotuner sets it

# Launch options the autotuner and the benchmark use (anything absent = the
# library's default).
TUNED_RANDOM = {"leaf": 64, "leaf_dc": True, "sweep_cols": 8, "wide_min": NO_WIDE, "fuse_few": 32}
TUNED_LARGE = {"leaf": 64, "leaf_dc": True, "sweep_cols": 16, "wide_min": 64, "wide_blocks": 256}
TUNED_TOEPLITZ = {"leaf": 64, "leaf_dc": True, "sweep_cols": 32, "wide_min": 32}
TUNED_BATCH = {"leaf": 8, "sweep_cols": 64, "wide_min": 64, "wide_blocks": 1024}
TUNED_GRAD = {"leaf": 8, "sweep_cols": 64, "wide_min": 1024, "wide_blocks": 256}
OPTIONS = ("leaf", "leaf_dc", "sweep_cols", "wide_min", "wide_blocks", "fuse_few")


def listed():
    return [
        # One small matrix out of the box, answer checked at once: a call inside
        # somebody's loop, where latency is everything.
        {"name": "small_default", "kind": "single", "family": "normal", "n": 300},
        # One matrix of ordinary, odd size out of the box.
        {"name": "mid_default", "kind": "single", "family": "uniform", "n": 10007},
        # The benchmark's own workload with its tuned options: solves in a loop
        # with kept buffers, status not read back.
        {"name": "uniform_65536", "kind": "loop", "family": "uniform", "n": 65536, **TUNED_RANDOM},
        # No deflation beyond symmetry (half of every merge stays): the O(n^2)
        # secular work of discretised differential operators.
        {"name": "toeplitz_65536", "kind": "loop", "family": "toeplitz", "n": 65536, **TUNED_TOEPLITZ},
        # The largest single matrix of the benchmark.
        {"name": "normal_262144", "kind": "loop", "family": "normal", "n": 262144, **TUNED_LARGE},
        # The benchmark's batch: many ragged problems in one call.
        {"name": "batch_4096", "kind": "batch", "B": 4096, "lo": 32, "hi": 4096, "shape": 1, **TUNED_BATCH},
        # Training step through one matrix with torch.autograd, out of the box.
        {"name": "autograd_8192", "kind": "autograd", "n": 8192},
        # Training step over a batch: checkpointing forward and reverse pass.
        {"name": "grad_256x1024", "kind": "grad", "B": 256, "lo": 1024, "hi": 1024, "shape": 2, **TUNED_GRAD},
        # Eigenvalues of a dense symmetric matrix (reduction and solve).
        {"name": "dense_4096", "kind": "dense", "n": 4096},
        # Gauss quadrature rules: nodes and first rows of ragged Jacobi matrices.
        {"name": "quadrature_32", "kind": "rows", "B": 32, "lo": 100, "hi": 1500, "shape": 3},
        # Chosen rows of one eigenvector matrix (a discrete polynomial transform).
        {"name": "selrows_3001", "kind": "selrows", "n": 3001, "m": 12},
        # A reducible matrix through the splitting driver, out of the box.
        {"name": "split_65536", "kind": "split", "n": 65536},
    ]


def _log(rng, lo, hi):
    return int(math.floor(math.exp(rng.uniform(math.log(lo), math.log(hi + 1)))))


def draw(rng):
    kind = rng.choice(["single", "single", "loop", "loop", "loop", "batch", "autograd", "grad", "dense", "rows",
                       "selrows", "split"])
    if kind == "single":
        return {"kind": kind, "family": rng.choice(["uniform", "normal", "clustered", "wilkinson"]),
                "n": _log(rng, 32, 65536)}
    if kind == "loop":
        family = rng.choice(["uniform", "normal", "toeplitz", "clustered", "wilkinson"])
        if family == "toeplitz":
            return {"kind": kind, "family": family, "n": _log(rng, 1000, 65536), **TUNED_TOEPLITZ}
        n = _log(rng, 4096, 262144)
        return {"kind": kind, "family": family, "n": n, **(TUNED_RANDOM if n <= 65536 else TUNED_LARGE)}
    if kind in ("batch", "grad", "rows"):
        hi = _log(rng, 64, 4096 if kind == "batch" else 1500)
        most = {"batch": 3000000, "grad": 262144, "rows": 40000}[kind] // hi
        opts = {"batch": TUNED_BATCH, "grad": TUNED_GRAD, "rows": {}}[kind]
        return {"kind": kind, "B": _log(rng, 4, max(8, min(4096, most))), "lo": min(hi, 32), "hi": hi,
                "shape": rng.randrange(1 << 20), **opts}
    if kind == "autograd":
        return {"kind": kind, "n": _log(rng, 256, 8192)}
    if kind == "dense":
        return {"kind": kind, "n": _log(rng, 128, 4000)}
    if kind == "selrows":
        return {"kind": kind, "n": _log(rng, 100, 3001), "m": rng.randint(1, 16)}
    return {"kind": kind, "n": _log(rng, 4096, 65536)}


def _sizes(case):
    """Ragged problem sizes of a batch, log-uniform in [lo, hi]: part of the case, not of its inputs."""
    rng = random.Random(case["shape"])
    return [min(case["hi"], _log(rng, case["lo"], case["hi"])) for _ in range(case["B"])]


def _offsets(sizes):
    offs = [0]
    for s in sizes:
        offs.append(offs[-1] + s)
    return offs


def _jacobi(n, a, b):
    """Recurrence matrix of the Jacobi polynomials P^(a,b), a, b > 0: (diagonal, off-diagonal)."""
    k = np.arange(n, dtype=np.float64)
    s = 2.0 * k + a + b
    d = (b * b - a * a) / (s * (s + 2.0))
    j = k[1:]
    t = 2.0 * j + a + b
    e = np.sqrt(4.0 * j * (j + a) * (j + b) * (j + a + b) / (t * t * (t + 1.0) * (t - 1.0)))
    return d, e


def _host_inputs(case, seed):
    """The pass's inputs as numpy arrays, from the seed alone."""
    g = np.random.default_rng([2605, seed])
    kind = case["kind"]
    if kind in ("single", "loop"):
        n, family = case["n"], case["family"]
        if family == "uniform":
            return g.uniform(-1.0, 1.0, n), g.uniform(-1.0, 1.0, n - 1)
        if family == "normal":
            return g.standard_normal(n), g.standard_normal(n - 1)
        if family == "toeplitz":
            return np.full(n, g.uniform(1.0, 3.0)), np.full(n - 1, -g.uniform(0.5, 1.5))
        if family == "clustered":
            scale = g.uniform(0.5, 2.0)
            return scale * 10.0 ** (-8.0 + 8.0 * np.arange(n) / max(n - 1, 1)), 1e-6 * g.uniform(0.0, 1.0, n - 1)
        scale = g.uniform(0.5, 2.0)  # wilkinson
        return scale * np.abs(np.arange(n) - (n - 1) / 2.0), np.full(n - 1, scale)
    if kind in ("batch", "grad"):
        n = sum(_sizes(case))
        return g.uniform(-1.0, 1.0, n), g.uniform(-1.0, 1.0, n), g.standard_normal(n)
    if kind == "autograd":
        n = case["n"]
        return g.uniform(-1.0, 1.0, n), g.uniform(-1.0, 1.0, n - 1), g.standard_normal(n)
    if kind == "rows":
        ds, es = [], []
        for n in _sizes(case):
            d, e = _jacobi(n, *g.uniform(0.1, 2.0, 2))
            ds.append(d)
            es.append(np.append(e, 0.0))
        return np.concatenate(ds), np.concatenate(es)
    if kind == "selrows":
        d, e = _jacobi(case["n"], *g.uniform(0.1, 2.0, 2))
        return d, e, g.integers(0, case["n"], case["m"])
    if kind == "split":
        n = case["n"]
        e = g.uniform(-1.0, 1.0, n - 1)
        e[g.choice(n - 1, n // 97, replace=False)] = 0.0
        return g.uniform(-1.0, 1.0, n), e
    raise ValueError(kind)


def _dense(case, seed):
    g = torch.Generator(device="cuda").manual_seed(2605 + 7919 * seed)
    A = torch.randn(case["n"], case["n"], dtype=torch.float64, device="cuda", generator=g)
    return (A + A.T) * (0.5 / math.sqrt(case["n"]))


def prepare(case, seed):
    kind = case["kind"]
    opts = {k: case[k] for k in OPTIONS if case.get(k) is not None}
    if kind == "dense":
        return {"kind": kind, "A": _dense(case, seed)}
    host = _host_inputs(case, seed)
    st = {"kind": kind, "opts": opts}
    st["d"], st["e"] = (torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in host[:2])
    n = st["d"].numel()
    if kind in ("batch", "grad", "rows"):
        st["offsets"] = _offsets(_sizes(case))
    if kind in ("autograd", "grad"):
        st["w"] = torch.from_numpy(host[2]).cuda()
    if kind == "autograd":
        st["d"].requires_grad_()
        st["e"].requires_grad_()
    if kind == "selrows":
        st["rows"] = [int(r) for r in host[2]]
    if kind in ("loop", "batch", "grad"):  # a solve loop keeps its buffers
        B = len(st["offsets"]) - 1 if "offsets" in st else 1
        st["out"] = torch.empty(n, dtype=torch.float64, device="cuda")
        nb = tde.workspace_bytes(n, B, opts.get("leaf"))
        if kind == "grad":
            nb = max(nb, int(tde.lib().tde_backward_workspace_bytes(n, B, None)))
            st["ckpt"] = torch.empty(tde.checkpoint_bytes(n, st["offsets"], opts.get("leaf"), opts.get("sweep_cols")),
                                     dtype=torch.uint8, device="cuda")
            st["gd"], st["ge"] = (torch.zeros(n, dtype=torch.float64, device="cuda") for _ in range(2))
        st["ws"] = torch.empty(nb, dtype=torch.uint8, device="cuda")
    return st


def run(state):
    kind = state["kind"]
    if kind == "dense":
        return tde.dense_eigvals(state["A"])
    d, e, opts = state["d"], state["e"], state["opts"]
    if kind == "single":
        return tde.eigvals(d, e, **opts)
    if kind == "loop":
        return tde.eigvals(d, e, out=state["out"], workspace=state["ws"], check=False, **opts)
    if kind == "batch":
        return tde.eigvals_batched(d, e, state["offsets"], out=state["out"], workspace=state["ws"], check=False, **opts)
    if kind == "autograd":
        lam = tde.differentiable_eigvals(d, e)
        gd, ge = torch.autograd.grad((lam * state["w"]).sum(), (d, e))
        return {"lam": lam.detach(), "gd": gd, "ge": ge}
    if kind == "grad":
        lam, ckpt = tde.eigvals_ckpt(d, e, state["offsets"], out=state["out"], ckpt=state["ckpt"],
                                     workspace=state["ws"], check=False, **opts)
        gd, ge = tde.eigvals_backward(d, e, state["w"], ckpt, state["offsets"], workspace=state["ws"], check=False,
                                      gd=state["gd"], ge=state["ge"], **opts)
        return {"lam": lam, "gd": gd, "ge": ge}
    if kind == "rows":
        lam, qfirst, _ = tde.eigvals_rows(d, e, state["offsets"], **opts)
        return {"nodes": lam, "first": qfirst}
    if kind == "selrows":
        lam, Q = tde.eigvals_selrows(d, e, state["rows"], **opts)
        return {"lam": lam, "Q": Q}
    lam, blocks = tde.eigvals_split(d, e, **opts)
    return {"lam": lam, "blocks": blocks}


def work(case):
    """Bytes: inputs once, outputs once.  Operations: the dense reduction's
    4/3 n^3; on the tridiagonal side what any such tree has to spend, about 20
    operations (order, z, deflation test, parent rows) on every column at
    every level, and as much again on the way back where gradients are asked
    for."""
    kind = case["kind"]
    if kind == "dense":
        n = case["n"]
        return {"bytes": 8.0 * n * n + 8.0 * n, "flops": 4.0 / 3.0 * n ** 3}
    sizes = _sizes(case) if kind in ("batch", "grad", "rows") else [case["n"]]
    cols = float(sum(sizes))
    flops = sum(20.0 * n * max(1.0, math.log2(n)) for n in sizes)
    if kind in ("grad", "autograd"):
        return {"bytes": 48.0 * cols, "flops": 2.0 * flops}
    rows = {"rows": 1, "selrows": case.get("m", 0)}.get(kind, 0)
    return {"bytes": (24.0 + 8.0 * rows) * cols, "flops": flops * (1 + rows / 2)}


def _tridiagonal(d, e):
    return np.diag(d) + np.diag(e, 1) + np.diag(e, -1)


def exact(case, seed):
    kind = case["kind"]
    if kind == "dense":
        return np.linalg.eigvalsh(_dense(case, seed).cpu().numpy())
    if kind in ("single", "loop") and case["family"] == "toeplitz":
        n = case["n"]
        d, e = _host_inputs(case, seed)
        k = np.arange(n, 0, -1)  # a + 2 b cos(k pi / (n + 1)), b < 0 ascending
        return np.sort(d[0] + 2.0 * e[0] * np.cos(k * (np.pi / (n + 1))))
    sizes = _sizes(case) if kind in ("batch", "grad", "rows") else [case["n"]]
    vectors = kind in ("autograd", "grad", "rows", "selrows")
    if sum(float(n) ** 3 for n in sizes) > (3e10 if vectors else 6e10):
        return None
    host = _host_inputs(case, seed)
    lams, first, gds, ges, Q = [], [], [], [], None
    at = 0
    for n in sizes:
        d, e = host[0][at:at + n], host[1][at:at + n - 1]
        T = _tridiagonal(d, e)
        if not vectors:
            lams.append(np.linalg.eigvalsh(T))
        else:
            lam, V = np.linalg.eigh(T)
            V = V * np.where(V[0] < 0.0, -1.0, 1.0)
            lams.append(lam)
            if kind == "rows":
                first.append(V[0])
            elif kind == "selrows":
                Q = V[host[2]]
            else:
                w = host[2][at:at + n]
                gds.append((V * V) @ w)
                ges.append(2.0 * (V[:-1] * V[1:]) @ w)
                if kind == "grad":
                    ges.append(np.zeros(1))
        at += n
    lam = np.concatenate(lams)
    if kind in ("autograd", "grad"):
        return {"lam": lam, "gd": np.concatenate(gds), "ge": np.concatenate(ges)}
    if kind == "rows":
        return {"nodes": lam, "first": np.concatenate(first)}
    if kind == "selrows":
        return {"lam": lam, "Q": Q}
    if kind == "split":
        return {"lam": lam, "blocks": None}
    return lam
