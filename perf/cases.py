"""The workloads whose speed this framework is judged by, as a user's program runs them.

Every case goes through the package's public calls.  The sizes and parameters are those of the
benchmark's modes and of the tests: the N = 1e6 matvec, the 32-rhs modes, the compression-error
columns of the paper's Sec 6.2, evaluation at new points, batches, CG solves and the solve server.

A case is a dict of plain values; `kind` names the call:
  matvec  y = K~ x                       (n, d, r, kernel, ell, q, leaf, eta, nrhs, precision, ...)
  eval    y = K~(targets, sources) x     (the same, and m targets)
  batch   one batched matvec over `count` problems, replayed from a HIP graph
  solve   (K~ + lam I) alpha = f from alpha = 0
  serve   `count` solve requests through the server: tree, operator and CG of each request
Points are uniform in the box [0, k^-r], the inputs of the paper's setting.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

import paper_2402_09531_amd as dw

# the most entries N x M for which the dense 64-bit sums of exact() are formed (a few seconds)
_EXACT_ENTRIES = 4.0e11

_DEFAULTS = {"nrhs": 1, "precision": "fp64", "leaf": 128, "eta": 0.8, "weight_rule": "R1", "nodes": "cheb_leja",
             "cache_near": False}


def _full(case: dict) -> dict:
    return {**_DEFAULTS, **case}


def listed() -> list[dict]:
    return [
        # the smallest call: the N = 4096 workload of the quick start, bound by launches and latency
        dict(name="matvec_small_d4", kind="matvec", n=4096, d=4, r=2.0, kernel="matern32", ell=1.0, q=4.0, leaf=64),
        # the benchmark's headline: one FP64 matvec at N = 1e6, d = 20
        dict(name="matvec_1m_d20", kind="matvec", n=1_000_000, d=20, r=3.0, kernel="gaussian", ell=0.5, q=6.0),
        # the other full-size geometry, one rhs, in the FP32 mode
        dict(name="matvec_1m_d10_fp32", kind="matvec", n=1_000_000, d=10, r=2.0, kernel="matern32", ell=1.0, q=6.0,
             precision="fp32"),
        # many right-hand sides in the BF16 MFMA mode
        dict(name="matvec_1m_d20_r32_bf16", kind="matvec", n=1_000_000, d=20, r=3.0, kernel="gaussian", ell=0.5,
             q=6.0, nrhs=32, precision="bf16"),
        # 25 columns of K~ in the paper's compression-error study, b_k = k^-2 (a large index set, n_x near 100)
        dict(name="columns_r2", kind="matvec", n=100_000, d=20, r=2.0, kernel="exponential", ell=0.1156, q=8.0,
             eta=1.0, nrhs=25, weight_rule="R3", nodes="afp"),
        # the same study with the larger leaves that its small length scales ask for, b_k = k^-3
        dict(name="columns_r3_leaf256", kind="matvec", n=100_000, d=20, r=3.0, kernel="exponential", ell=0.039, q=8.0,
             eta=1.0, nrhs=25, leaf=256, weight_rule="R3", nodes="afp"),
        # an interpolant evaluated at new points
        dict(name="eval_300k", kind="eval", n=1_000_000, m=300_000, d=20, r=3.0, kernel="gaussian", ell=0.5, q=6.0),
        # several interpolants on the same sites evaluated at new points, a ragged number of them
        dict(name="eval_r8", kind="eval", n=100_003, m=50_001, d=10, r=2.0, kernel="matern32", ell=1.0, q=5.0, nrhs=8),
        # the batching workload: many independent problems of very different sizes per call
        dict(name="batch_48", kind="batch", count=48, n_lo=2000, n_hi=200_000, d_lo=8, d_hi=16, r=2.0,
             kernel="matern32", ell=1.0, q=5.0, spec=4),
        # a small CG solve: a few dozen iterations of small launches
        dict(name="solve_small_d4", kind="solve", n=4096, d=4, r=2.0, kernel="matern32", ell=1.0, q=4.0, leaf=64,
             lam=0.5, rtol=1e-8),
        # 32 systems at once, BF16 inner products with FP64 refinement
        dict(name="solve_200k_r32_bf16", kind="solve", n=200_000, d=20, r=3.0, kernel="gaussian", ell=0.5, q=6.0,
             nrhs=32, precision="bf16", lam=100.0, rtol=1e-8),
        # requests of the serving trace, from the points on the host to alpha on the host
        dict(name="serve_16", kind="serve", count=16, n_lo=1000, n_hi=100_000, d_lo=6, d_hi=24, lam=10.0, rtol=1e-8,
             spec=5),
    ]


def _log_uniform(rng: random.Random, lo: float, hi: float) -> int:
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random) -> dict:
    kind = rng.choice(["matvec", "matvec", "matvec_lp", "columns", "eval", "batch", "solve", "serve"])
    kernel, ell = rng.choice([("matern32", 1.0), ("gaussian", 0.5), ("exponential", 0.3)])
    d = rng.randint(4, 24)
    r = rng.choice([2.0, 3.0])
    q = float(rng.randint(4, 6))
    if kind in ("matvec", "matvec_lp"):
        n = _log_uniform(rng, 1000, 600_000)
        nrhs = rng.choice([1, 1, 1, rng.randint(2, 32)])
        c = dict(kind="matvec", n=n, d=d, r=r, kernel=kernel, ell=ell, q=q, nrhs=nrhs,
                 leaf=rng.choice([64, 100, 128, 128]))
        if nrhs > 1:
            c["n"] = min(n, 250_000)
        if kind == "matvec_lp":
            c["precision"] = rng.choice(["fp32", "bf16"])
            if nrhs > 1 and c["precision"] == "bf16":
                c["cache_near"] = rng.random() < 0.5
        return c
    if kind == "columns":
        r, sigma = rng.choice([(2.0, 0.1156), (2.0, 0.2851), (3.0, 0.039), (3.0, 0.2149), (4.0, 0.0188)])
        return dict(kind="matvec", n=_log_uniform(rng, 20_000, 100_000), d=20, r=r, kernel="exponential", ell=sigma,
                    q=8.0, eta=1.0, nrhs=rng.choice([1, rng.randint(2, 25), 25]), leaf=rng.choice([64, 128, 256]),
                    weight_rule="R3", nodes="afp")
    if kind == "eval":
        nrhs = rng.choice([1, 1, rng.randint(2, 16)])
        hi = 500_000 if nrhs == 1 else 60_000
        return dict(kind="eval", n=_log_uniform(rng, 4000, hi), m=_log_uniform(rng, 100, hi), d=d, r=r, kernel=kernel,
                    ell=ell, q=q, nrhs=nrhs)
    if kind == "batch":
        return dict(kind="batch", count=rng.randint(4, 48), n_lo=1000, n_hi=_log_uniform(rng, 4000, 200_000), d_lo=8,
                    d_hi=16, r=2.0, kernel="matern32", ell=1.0, q=5.0, spec=rng.randrange(1 << 20))
    if kind == "solve":
        n = _log_uniform(rng, 1000, 60_000)
        return dict(kind="solve", n=n, d=rng.randint(6, 24), r=r, kernel="matern32", ell=1.0, q=q,
                    nrhs=rng.choice([1, 1, rng.randint(2, 32)]), precision=rng.choice(["fp64", "fp32"]),
                    lam=max(10.0, n / 1000.0), rtol=1e-8)
    return dict(kind="serve", count=rng.randint(2, 16), n_lo=1000, n_hi=_log_uniform(rng, 2000, 60_000), d_lo=6,
                d_hi=24, lam=10.0, rtol=1e-8, spec=rng.randrange(1 << 20))


def _dim_weights(d: int, r: float) -> np.ndarray:
    return np.arange(1, d + 1, dtype=np.float64) ** (-float(r))


def _points(n: int, d: int, r: float, gen: torch.Generator) -> torch.Tensor:
    b = torch.from_numpy(_dim_weights(d, r)).cuda()
    return torch.rand((n, d), dtype=torch.float64, device="cuda", generator=gen) * b


def _batch_spec(c: dict) -> list[tuple[int, int]]:
    """(N, d) of each problem, fixed by the case."""
    rng = random.Random(c["spec"])
    return [(_log_uniform(rng, c["n_lo"], c["n_hi"]), rng.randint(c["d_lo"], c["d_hi"])) for _ in range(c["count"])]


def _serve_spec(c: dict) -> list[tuple[int, int, float, float]]:
    """(N, d, r, q) of each request, fixed by the case."""
    rng = random.Random(c["spec"])
    return [(_log_uniform(rng, c["n_lo"], c["n_hi"]), rng.randint(c["d_lo"], c["d_hi"]), rng.choice([2.0, 3.0]),
             float(rng.randint(4, 6))) for _ in range(c["count"])]


def _inputs(c: dict, seed: int) -> dict:
    """The points and vectors of a case (on the GPU; a request's on the host)."""
    gen = torch.Generator(device="cuda").manual_seed(seed)
    if c["kind"] == "serve":
        reqs = []
        for i, (n, d, r, q) in enumerate(_serve_spec(c)):
            rng = np.random.default_rng(1_000_003 * seed + i)
            b = _dim_weights(d, r)
            X = rng.random((n, d)) * b
            reqs.append((X, b, np.sin(X.sum(axis=1)), q))
        return {"requests": reqs}
    if c["kind"] == "batch":
        probs = []
        for n, d in _batch_spec(c):
            X = _points(n, d, c["r"], gen)
            probs.append((X, torch.randn((n, 1), dtype=torch.float64, device="cuda", generator=gen)))
        return {"problems": probs}
    X = _points(c["n"], c["d"], c["r"], gen)
    out = {"X": X}
    if c["kind"] == "solve":
        # one data function per column, smooth in the points
        k = torch.arange(1, c["nrhs"] + 1, dtype=torch.float64, device="cuda")
        out["f"] = torch.sin(X.sum(dim=1, keepdim=True) * (0.5 + 0.5 * k)[None, :]).contiguous()
        return out
    out["x"] = torch.randn((c["n"], c["nrhs"]), dtype=torch.float64, device="cuda", generator=gen)
    if c["kind"] == "eval":
        out["T"] = _points(c["m"], c["d"], c["r"], gen)
    return out


def _operator(c: dict, X: torch.Tensor, d: int):
    tree = dw.build_tree(X, _dim_weights(d, c["r"]), c["leaf"], c["eta"])
    return dw.fmm_create(tree, c["kernel"], c["ell"], c["q"], precision=c["precision"], max_nrhs=c["nrhs"],
                         weight_rule=c["weight_rule"], nodes=c["nodes"], cache_near=c["cache_near"])


def prepare(case: dict, seed: int) -> dict:
    c = _full(case)
    s = {"case": c, **_inputs(c, seed)}
    if c["kind"] == "serve":
        s["server"] = dw.Server(64 << 30, max_active=64, check_every=1)
    elif c["kind"] == "batch":
        ops = [_operator(c, X, X.shape[1]) for X, _ in s["problems"]]
        s["batch"] = dw.batch_create(ops, graph=True)
        s["xs"] = [x for _, x in s["problems"]]
        s["ys"] = [torch.empty_like(x) for x in s["xs"]]
    else:
        s["op"] = _operator(c, s["X"], c["d"])
        if c["kind"] == "matvec":
            s["y"] = torch.empty_like(s["x"])
        elif c["kind"] == "eval":
            s["eval"] = dw.eval_create(s["op"], s["T"])
            s["y"] = torch.empty((c["m"], c["nrhs"]), dtype=torch.float64, device="cuda")
    return s


def run(s: dict):
    c = s["case"]
    if c["kind"] == "matvec":
        dw.fmm_matvec(s["op"], s["x"], s["y"])
        return s["y"]
    if c["kind"] == "eval":
        dw.eval_apply(s["eval"], s["x"], s["y"])
        return s["y"]
    if c["kind"] == "batch":
        dw.batch_matvec(s["batch"], s["xs"], s["ys"])
        return s["ys"]
    if c["kind"] == "solve":
        alpha = torch.zeros_like(s["f"])
        dw.fmm_solve(s["op"], c["lam"], s["f"], alpha, c["rtol"], 400)
        return alpha
    srv = s["server"]
    ids = [srv.submit(X, b, f, 128, 0.8, "matern32", 1.0, q, c["lam"], c["rtol"], 400)
           for X, b, f, q in s["requests"]]
    got = {}
    while len(got) < len(ids):
        srv.tick()
        for rid in srv.finished():
            got[rid] = srv.result(rid)[0]
    return [got[rid] for rid in ids]


def _near_per_point(n: int, leaf: int) -> float:
    """About how many sources a point meets in the nearfield (1.98e4 at N = 1e6, d = 20, leaf 128)."""
    return float(min(n, 155 * leaf))


def work(case: dict) -> dict:
    """Points, vectors and results once; the nearfield entries (each unordered pair evaluated once in a
    square operator) at 3 d + 6 flops, and two flops per applied entry and rhs."""
    c = _full(case)

    def matvec(n, d, nrhs, m=None):
        t = n if m is None else m
        e = t * _near_per_point(n, c["leaf"])
        flops = e * ((3 * d + 6) * (0.5 if m is None else 1.0) + 2 * nrhs)
        return 8.0 * (n * d + n * nrhs + t * nrhs + (0 if m is None else m * d)), flops

    if c["kind"] == "matvec":
        b, f = matvec(c["n"], c["d"], c["nrhs"])
    elif c["kind"] == "eval":
        b, f = matvec(c["n"], c["d"], c["nrhs"], c["m"])
    elif c["kind"] == "batch":
        parts = [matvec(n, d, 1) for n, d in _batch_spec(c)]
        b, f = sum(p[0] for p in parts), sum(p[1] for p in parts)
    elif c["kind"] == "solve":
        its = 40  # about the iterations such a solve takes
        b, f = matvec(c["n"], c["d"], c["nrhs"])
        f *= its
    else:
        parts = [matvec(n, d, 1) for n, d, _, _ in _serve_spec(c)]
        b, f = sum(p[0] for p in parts), 40 * sum(p[1] for p in parts)
    return {"bytes": b, "flops": f}


def _dense(kernel: str, ell: float, T: torch.Tensor, X: torch.Tensor, x: torch.Tensor) -> torch.Tensor:
    """sum_j K(t_i, x_j) x_j in 64 bits, a block of targets at a time."""
    y = torch.empty((T.shape[0], x.shape[1]), dtype=torch.float64, device=X.device)
    c = X.mean(dim=0)
    Xc, xn = X - c, ((X - c) ** 2).sum(dim=1)
    step = max(1, int(2.0e8 // X.shape[0]))
    for i in range(0, T.shape[0], step):
        t = T[i:i + step] - c
        r2 = torch.addmm(xn[None, :] + (t * t).sum(dim=1, keepdim=True), t, Xc.t(), alpha=-2.0).clamp_(min=0.0)
        if kernel == "gaussian":
            K = r2.mul_(-1.0 / ell).exp_()
        elif kernel == "exponential":
            K = r2.sqrt_().mul_(-1.0 / ell).exp_()
        else:
            s = r2.sqrt_().mul_(math.sqrt(3.0) / ell)
            K = (1.0 + s) * torch.exp(-s)
        y[i:i + step] = K @ x
    return y


def exact(case: dict, seed: int):
    """The dense sums K x that the operator approximates (to its interpolation error); None for
    solutions of K~ alpha = f, which are those of the approximate operator, and for sizes too large."""
    c = _full(case)
    if c["kind"] in ("solve", "serve"):
        return None
    if c["kind"] == "batch":
        if sum(float(n) * n for n, _ in _batch_spec(c)) > _EXACT_ENTRIES:
            return None
        s = _inputs(c, seed)
        return [_dense(c["kernel"], c["ell"], X, X, x) for X, x in s["problems"]]
    if float(c["n"]) * c.get("m", c["n"]) > _EXACT_ENTRIES:
        return None
    s = _inputs(c, seed)
    return _dense(c["kernel"], c["ell"], s["T"] if c["kind"] == "eval" else s["X"], s["X"], s["x"])
