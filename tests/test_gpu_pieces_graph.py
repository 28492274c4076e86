"""Large leaves and evaluation from a captured graph: under capture everything stays on one stream and the
nearfield of pieces adds the farfield itself; the eager matvec runs the farfield beside it and adds it
afterwards.  Same bits, over several replays with eager work and synchronisations between them; every
kernel of the pieces form (in range, split, clamped and past the bound of the Gram form), one rhs, one rhs
tile and two, the wide coupling.
"""
import gc

import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2402_09531_amd as dw  # noqa: E402
from paper_2402_09531_amd import workloads as W  # noqa: E402


@pytest.mark.parametrize("nrhs", [1, 5, 20])
@pytest.mark.parametrize("kind,ell,d,q", [
    ("matern32", 1.0, 8, 4), ("matern32", 0.02, 8, 4), ("matern32", 1e-3, 3, 4), ("exponential", 0.3, 8, 4),
    ("exponential", 1e-3, 8, 4), ("gaussian", 0.5, 8, 4), ("gaussian", 2e-3, 8, 4), ("gaussian", 0.5, 6, 10),
])
def test_graph_equals_eager(kind, ell, d, q, nrhs):
    n, m = 6000, 1501
    X, b = W.points(n, d, 2.0, 63), W.dim_weights(d, 2.0)
    op = dw.fmm_create(dw.build_tree(torch.from_numpy(X).cuda(), b, 256, 0.8), kind, ell, q, max_nrhs=nrhs)
    ev = dw.eval_create(op, torch.from_numpy(W.points(m, d, 2.0, 64)).cuda())
    print(f"[pieces graph] {kind} ell={ell:g} d={d} n_x={op.nx} nrhs={nrhs}", flush=True)
    rng = np.random.default_rng(65)
    x, x2 = (torch.from_numpy(rng.standard_normal((n, nrhs))).cuda() for _ in range(2))
    y, y2, yg = (torch.empty_like(x) for _ in range(3))
    z, zg = (torch.empty((m, nrhs), dtype=torch.float64, device="cuda") for _ in range(2))
    dw.fmm_matvec(op, x, y)
    dw.eval_apply(ev, x, z)
    torch.cuda.synchronize()
    gc.collect()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, capture_error_mode="thread_local"):
        dw.fmm_matvec(op, x, yg)
        dw.eval_apply(ev, x, zg)
    for rep in range(3):
        yg.zero_()
        zg.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(yg, y) and torch.equal(zg, z), rep
        dw.fmm_matvec(op, x2, y2)
        torch.cuda.synchronize()
