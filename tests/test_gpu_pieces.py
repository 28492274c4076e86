"""FP64 matrix-core paths of large leaves, several-rhs evaluation and large index sets, against the oracle.

Leaves above 128 points run the nearfield in pieces of at most 128 targets, evaluation with several
rhs (or large target leaves) runs the same kernel over two trees, and index sets above 64 nodes
(above 32 with several rhs) run the wide coupling.  The sizes sit at the edges: one point over a
piece, a piece of one row tile, the largest leaf, 1 / 16 / 17 / 32 rhs, 3 to 8 node tiles, a last
node tile with one node.  Bound: the 1e-12 of every FP64 parity test (the exponential kernel at
coincident points included: its distances there are taken from the coordinates).
"""
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2402_09531_amd as dw  # noqa: E402
from paper_2402_09531_amd import workloads as W  # noqa: E402

TOL = 1e-12


def say(*a):
    print(*a, flush=True)
    sys.stdout.flush()


def rel(a, b):
    return np.linalg.norm(a - b) / np.linalg.norm(b)


SQUARE = [
    # n, d, r, kernel, ell, q, leaf, nrhs, precision, node tiles
    (129, 4, 2.0, "exponential", 0.3, 4, 129, 1, "fp64", None),      # one leaf, one point over a piece
    (4000, 5, 2.0, "gaussian", 0.5, 4, 250, 1, "fp64", None),        # split Gaussian, one rhs
    (5001, 7, 2.0, "exponential", 0.3, 4, 313, 16, "fp64", None),    # three pieces
    (6000, 10, 2.0, "matern32", 1.0, 4, 200, 17, "fp64", None),
    (4100, 2, 1.0, "exponential", 0.3, 3, 1024, 2, "fp64", None),    # the largest leaves; d = 2: close points
    (3000, 20, 3.0, "gaussian", 2e-3, 4, 256, 32, "fp64", None),     # direct Gaussian
    (4000, 30, 3.0, "matern32", 1.0, 4, 250, 5, "fp64", None),
    (3000, 6, 2.0, "matern32", 1.0, 4, 190, 3, "bf16", None),        # FP64 nearfield in every mode
    (6000, 20, 3.0, "gaussian", 0.5, 12, 64, 1, "fp64", 7),
    (6000, 6, 2.0, "exponential", 0.3, 8, 64, 25, "fp64", 4),
    (6000, 3, 2.0, "matern32", 1.0, 8, 64, 3, "fp64", 3),
    (5000, 6, 2.0, "matern32", 1.0, 10, 50, 17, "fp64", 8),
]


@pytest.mark.parametrize("case", SQUARE, ids=[f"{c[3]}_n{c[0]}_d{c[1]}_q{c[5]}_leaf{c[6]}_r{c[7]}" for c in SQUARE])
def test_square(orc, case):
    n, d, r, kind, ell, q, leaf, nrhs, prec, tiles = case
    X, b = W.points(n, d, r, 40 + n), W.dim_weights(d, r)
    x = np.random.default_rng(41 + n).standard_normal((n, nrhs))
    tree = dw.build_tree(torch.from_numpy(X).cuda(), b, leaf, 0.8)
    op = dw.fmm_create(tree, kind, ell, q, max_nrhs=nrhs, precision=prec)
    say(f"[pieces] {case} n_x={op.nx} far blocks {tree.nF} near {tree.nN}")
    if tiles is not None:
        assert (op.nx + 15) // 16 == tiles and tree.nF > 0
    xd = torch.from_numpy(x).cuda()
    yd, ys = torch.empty_like(xd), torch.empty_like(xd)
    dw.fmm_matvec(op, xd, yd, parts=3 if prec == "fp64" else 1, precision=prec)
    dw.fmm_matvec(op, xd, ys, parts=3 if prec == "fp64" else 1, precision=prec)
    torch.cuda.synchronize()
    assert torch.equal(yd, ys)
    yr = orc.Plan(X, b, leaf, 0.8, kind, ell, q).matvec(x, parts=3 if prec == "fp64" else 1)
    e = rel(yd.cpu().numpy(), yr)
    say(f"   relative error vs oracle {e:.2e}")
    assert e <= TOL


EVAL = [
    # n, m, d, r, kernel, ell, q, leaf, nrhs, targets = sources
    (6000, 2500, 6, 2.0, "exponential", 0.3, 4, 64, 8, False),
    (5000, 5000, 7, 2.0, "exponential", 0.3, 4, 100, 3, True),       # coincident points
    (5000, 20011, 10, 2.0, "matern32", 1.0, 4, 100, 17, False),      # target leaves above 128
    (5000, 30000, 4, 2.0, "gaussian", 0.5, 4, 100, 1, False),        # the same, one rhs, split Gaussian
    (4000, 33, 20, 3.0, "gaussian", 0.5, 6, 128, 32, False),
    (6000, 1500, 6, 2.0, "matern32", 1.0, 10, 50, 5, False),         # wide coupling
    (6000, 1500, 20, 3.0, "gaussian", 0.5, 12, 64, 1, False),
]


@pytest.mark.parametrize("case", EVAL, ids=[f"{c[4]}_n{c[0]}_m{c[1]}_d{c[2]}_q{c[6]}_r{c[8]}" for c in EVAL])
def test_eval(orc, case):
    n, m, d, r, kind, ell, q, leaf, nrhs, same = case
    X, b = W.points(n, d, r, 60 + n), W.dim_weights(d, r)
    T = X.copy() if same else W.points(m, d, r, 61 + m) * 1.05
    x = np.random.default_rng(62 + n).standard_normal((n, nrhs))
    tree = dw.build_tree(torch.from_numpy(X).cuda(), b, leaf, 0.8)
    op = dw.fmm_create(tree, kind, ell, q, max_nrhs=nrhs)
    ev = dw.eval_create(op, torch.from_numpy(T).cuda())
    say(f"[pieces] eval {case} n_x={op.nx} far blocks {ev.nF} near {ev.nN}")
    xd = torch.from_numpy(x).cuda()
    yd = torch.empty((m, nrhs), dtype=torch.float64, device="cuda")
    dw.eval_apply(ev, xd, yd)
    torch.cuda.synchronize()
    P = orc.Plan(X, b, leaf, 0.8, kind, ell, q)
    e = rel(yd.cpu().numpy(), orc.Eval(P, T).apply(x))
    say(f"   relative error vs oracle {e:.2e}")
    assert e <= TOL


@pytest.mark.parametrize("n,d,q,leaf,nrhs", [(33000, 6, 4, 4, 2), (33000, 6, 4, 4, 17), (9000, 6, 8, 8, 16), (5000, 3, 6, 2, 32)])
def test_several_rhs_transfers(n, d, q, leaf, nrhs):
    """Moments and locals of every cluster: each column of a several-rhs pass (MFMA, levels joined in
    groups) against the one-rhs pass of that column.  Both sum the same products in FP64: within
    n_x J eps of the largest value, 128 * 14 * 1.1e-16 = 2e-13, taken per array."""
    X, b = W.points(n, d, 2.0, 80 + n), W.dim_weights(d, 2.0)
    x = np.random.default_rng(81 + n).standard_normal((n, nrhs))
    tree = dw.build_tree(torch.from_numpy(X).cuda(), b, leaf, 0.8)
    op = dw.fmm_create(tree, "matern32", 1.0, q, max_nrhs=nrhs)
    say(f"[pieces] transfers n={n} J={tree.J} n_x={op.nx} nrhs={nrhs}")
    xd = torch.from_numpy(x).cuda()
    yd = torch.empty_like(xd)
    dw.fmm_matvec(op, xd, yd, parts=2)
    m, l = op.moments(nrhs)
    for r in {0, nrhs // 2, nrhs - 1}:
        x1 = xd[:, r:r + 1].contiguous()
        y1 = torch.empty_like(x1)
        dw.fmm_matvec(op, x1, y1, parts=2)
        m1, l1 = op.moments(1)
        lv = slice((1 << min_far_level(tree)) - 1, None)
        assert np.abs(m[lv, :, r] - m1[lv, :, 0]).max() <= 2e-13 * np.abs(m1).max()
        assert np.abs(l[lv, :, r] - l1[lv, :, 0]).max() <= 2e-13 * np.abs(l1).max()


def min_far_level(tree):
    c = int(np.flatnonzero(np.diff(tree.host()["Fptr"]))[0])
    return (c + 1).bit_length() - 1
