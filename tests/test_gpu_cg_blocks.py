"""One-rhs CG at the edges of its blocks: one workgroup for the whole iteration (n <= 4096), two and more
blocks finished by the last one, rows read eight at a time with every remainder, and the state read one
iteration late for small problems.  The solution's residual, re-measured by a matvec, is the tolerance
it stopped at (1e-8, and 1e-12 of slack for the recurrence's own drift); a progress callback (state read
in every iteration) and checks every third iteration leave the same bits, and so does a batch.
"""
import sys

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2402_09531_amd as dw  # noqa: E402
from paper_2402_09531_amd import workloads as W  # noqa: E402


@pytest.mark.parametrize("n", [1, 255, 2049, 4096, 4097, 8200, 30001])
def test_cg_blocks(n):
    print(f"[cg] n={n}", flush=True)
    sys.stdout.flush()
    d, lam = 6, 10.0
    X, b = W.points(n, d, 2.0, 90 + n), W.dim_weights(d, 2.0)
    Xd = torch.from_numpy(X).cuda()
    f = torch.from_numpy(np.sin(X.sum(axis=1))[:, None].copy()).cuda()
    got = []
    for kw in ({}, {"progress": lambda it, rr: None}, {"check_every": 3}):
        op = dw.fmm_create(dw.build_tree(Xd, b, 64, 0.8), "matern32", 1.0, 5, **kw)
        a = torch.zeros_like(f)
        info = dw.fmm_solve(op, lam, f, a, 1e-8, 400)[0]
        assert info["status"] == 0 and info["iters"] > 0
        got.append((a, info["iters"], op))
    a, it, op = got[0]
    assert all(torch.equal(a, o[0]) and it == o[1] for o in got[1:])
    y = torch.empty_like(a)
    dw.fmm_matvec(op, a, y)
    res = float(torch.linalg.norm(f - y - lam * a) / torch.linalg.norm(f))
    assert res <= 1e-8 + 1e-12, res
    # capped: no step past max_iter
    a2 = torch.zeros_like(f)
    assert dw.fmm_solve(op, lam, f, a2, 1e-300, 2)[0]["iters"] <= 2
    a3 = torch.zeros_like(f)
    info = dw.batch_solve(dw.batch_create([op]), lam, [f], [a3], 1e-8, 400, check_every=2)[0]
    assert info["iters"] == it and torch.equal(a, a3)
