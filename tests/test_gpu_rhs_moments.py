"""Moments and farfield evaluation of several rhs on FP64 MFMA, against the oracle.

Edges: 2 / 15 / 16 / 17 / 32 rhs (one and two rhs tiles, a thread group that does not divide 256),
leaves of one point, of a point over a 4-, 16- and 32-point step and of 64 and 128 points, index sets
around a 4- and a 16-node step.  Bound: the 1e-12 of every FP64 parity test.

The CG vector passes: four steps against the same four steps in torch, with and without
a ridge, rows that do not fill a block's steps.  The sums' rounding (1e-16 sqrt(n) of their terms) enters
each step's two ratios; four steps on a random right-hand side keep it under 1e-10.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2402_09531_amd as dw  # noqa: E402
from paper_2402_09531_amd import workloads as W  # noqa: E402

CASES = [
    # n, d, r, q, leaf, nrhs
    (600, 2, 1.0, 3, 1, 2),
    (2100, 3, 1.5, 4, 17, 15),
    (4200, 4, 2.0, 5, 33, 16),
    (4096, 6, 2.0, 6, 64, 17),
    (8191, 8, 2.0, 3, 128, 32),
    (5000, 20, 3.0, 6, 49, 25),
]


@pytest.mark.parametrize("case", CASES, ids=["n%d_d%d_r%g_q%d_leaf%d_r%d" % c for c in CASES])
def test_columns(orc, case):
    n, d, r, q, leaf, nrhs = case
    X, b = W.points(n, d, r, 70 + n), W.dim_weights(d, r)
    x = np.random.default_rng(71 + n).standard_normal((n, nrhs))
    tree = dw.build_tree(torch.from_numpy(X).cuda(), b, leaf, 0.8)
    op = dw.fmm_create(tree, "matern32", 1.0, q, max_nrhs=nrhs)
    print(f"[moments] {case} n_x={op.nx} far blocks {tree.nF}", flush=True)
    xd = torch.from_numpy(x).cuda()
    yd = torch.empty_like(xd)
    dw.fmm_matvec(op, xd, yd)
    torch.cuda.synchronize()
    ref = orc.Plan(X, b, leaf, 0.8, "matern32", 1.0, q).matvec(x)
    assert np.linalg.norm(yd.cpu().numpy() - ref) <= 1e-12 * np.linalg.norm(ref)


@pytest.mark.parametrize("n,nrhs", [(1, 2), (257, 3), (1024, 32), (4099, 17), (20011, 25)])
@pytest.mark.parametrize("lam", [0.0, 10.0])
def test_cg_steps(n, nrhs, lam):
    d = 4
    X, b = W.points(n, d, 2.0, 80 + n), W.dim_weights(d, 2.0)
    f = torch.from_numpy(np.random.default_rng(81 + n).standard_normal((n, nrhs))).cuda()
    op = dw.fmm_create(dw.build_tree(torch.from_numpy(X).cuda(), b, 64, 0.8), "matern32", 1.0, 4, max_nrhs=nrhs)
    steps = min(4, n)
    print(f"[cg steps] n={n} nrhs={nrhs} lambda={lam}", flush=True)
    a = torch.zeros_like(f)
    info = dw.fmm_solve(op, lam, f, a, 1e-300, steps)
    assert all(i["iters"] == steps for i in info)
    x, r, q = torch.zeros_like(f), f.clone(), torch.empty_like(f)
    p, rr = r.clone(), (r * r).sum(0)
    for _ in range(steps):
        dw.fmm_matvec(op, p, q)
        q += lam * p
        s = rr / (p * q).sum(0)
        x += s * p
        r -= s * q
        new = (r * r).sum(0)
        p = r + (new / rr) * p
        rr = new
    assert float(torch.linalg.norm(a - x)) <= 1e-10 * float(torch.linalg.norm(x))
