"""Clouds away from the origin: every coupling (one rhs and several, small and large index sets, matvec
and evaluation, FP64 and FP32) on the cloud shifted by 10 and 1e4 in each coordinate.

The kernel depends on differences only, and the oracle takes them from the shifted coordinates, so the
bounds are those of clouds at the origin: 1e-12 in FP64 as in every parity test; in FP32 the farfield
alone against the oracle's, 1e-5 (the moments' and locals' rounding, 6e-8 sqrt(n_x), with the
distances' 2^-24 times the ratio of the cloud's norm to a far block's distance, about 50).
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2402_09531_amd as dw  # noqa: E402
from paper_2402_09531_amd import workloads as W  # noqa: E402

CASES = [
    # n, d, r, kernel, ell, q, nrhs
    (4000, 6, 2.0, "matern32", 1.0, 4, 1),       # up to 64 nodes, one rhs
    (4000, 6, 2.0, "matern32", 1.0, 4, 5),       # up to 32 nodes, several rhs
    (4000, 20, 3.0, "gaussian", 0.5, 12, 1),     # above 64 nodes
    (4000, 6, 2.0, "exponential", 0.3, 8, 5),    # above 32 nodes, one rhs tile
    (4000, 6, 2.0, "exponential", 0.3, 8, 20),   # the same, two
]
IDS = ["%s_d%d_q%d_r%d" % (c[3], c[1], c[5], c[6]) for c in CASES]


def rel(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


def problem(case, off, **kw):
    n, d, r, kind, ell, q, nrhs = case
    X, b = W.points(n, d, r, 1) + off, W.dim_weights(d, r)
    x = np.random.default_rng(2).standard_normal((n, nrhs))
    tree = dw.build_tree(torch.from_numpy(X).cuda(), b, 64, 0.8)
    assert tree.nF > 0
    return X, b, x, dw.fmm_create(tree, kind, ell, q, max_nrhs=nrhs, **kw)


@pytest.mark.parametrize("off", [0.0, 10.0, 1e4])
@pytest.mark.parametrize("case", CASES, ids=IDS)
def test_fp64(orc, case, off):
    print(f"[offset] {case} {off:g}", flush=True)
    n, d, r, kind, ell, q, nrhs = case
    X, b, x, op = problem(case, off)
    xd = torch.from_numpy(x).cuda()
    yd = torch.empty_like(xd)
    dw.fmm_matvec(op, xd, yd)
    P = orc.Plan(X, b, 64, 0.8, kind, ell, q)
    e = rel(yd.cpu().numpy(), P.matvec(x))
    T = W.points(1500, d, r, 3) + off
    zd = torch.empty((1500, nrhs), dtype=torch.float64, device="cuda")
    dw.eval_apply(dw.eval_create(op, torch.from_numpy(T).cuda()), xd, zd)
    e2 = rel(zd.cpu().numpy(), orc.Eval(P, T).apply(x))
    print(f"   n_x={op.nx} matvec {e:.1e} evaluation {e2:.1e}", flush=True)
    assert e <= 1e-12 and e2 <= 1e-12


@pytest.mark.parametrize("off", [0.0, 10.0, 1e4])
@pytest.mark.parametrize("nrhs", [1, 5])
def test_fp32(orc, nrhs, off):
    print(f"[offset] fp32 {nrhs} {off:g}", flush=True)
    case = (4000, 6, 2.0, "matern32", 1.0, 4, nrhs)
    X, b, x, op = problem(case, off, precision="fp32")
    xd = torch.from_numpy(x).cuda()
    yd = torch.empty_like(xd)
    dw.fmm_matvec(op, xd, yd, parts=2, precision="fp32")
    e = rel(yd.cpu().numpy(), orc.Plan(X, b, 64, 0.8, "matern32", 1.0, 4).matvec(x, parts=2))
    print(f"   {e:.1e}", flush=True)
    assert e <= 1e-5
