"""Close points in the FP64 nearfield of pieces (large leaves, evaluation), against sums in extended precision.

One leaf holds everything (no farfield), every point has a partner at a fraction of the length scale and
some coincide, and the length scale runs from the size of the cloud to a thousandth of it: the kernels in
range, the same past the bound of their Gram form, and the clamped ones, d up to 4 and beyond, one row
tile of rhs and two, the largest tile in LDS (d = 27, 32 rhs).

Bounds per entry of order one, rho the cloud's diameter over the length scale, eps = 1.1e-16: Matern and
the split Gaussian in range 1.5 eps rho^2 under 1e-13 (rho <= 24, rho^2 <= 300), past it 8e-15 from the
threshold of 1e-2 and 1e-15 from the differences (d <= 4); the exponential 18 eps at any rho (the largest
value of eps rho exp(-rho / 10) / 0.2).  A row holds two or three such entries beside 300 small ones:
three times that.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2402_09531_amd as dw  # noqa: E402
from paper_2402_09531_amd import workloads as W  # noqa: E402

ELL = {"matern32": (0.1, 0.01, 1e-3), "exponential": (0.1, 0.01, 1e-3), "gaussian": (0.05, 3e-3, 1e-5)}


def dense(kind, ell, T, X, x):
    r2 = np.zeros((len(T), len(X)), dtype=np.longdouble)
    for k in range(X.shape[1]):
        r2 += (T[:, k].astype(np.longdouble)[:, None] - X[:, k].astype(np.longdouble)[None]) ** 2
    ell = np.longdouble(ell)
    if kind == "gaussian":
        K = np.exp(-r2 / ell)
    elif kind == "exponential":
        K = np.exp(-np.sqrt(r2) / ell)
    else:
        s = np.sqrt(np.longdouble(3) * r2) / ell
        K = (1 + s) * np.exp(-s)
    return (K @ x.astype(np.longdouble)).astype(np.float64)


@pytest.mark.parametrize("kind", ["matern32", "exponential", "gaussian"])
@pytest.mark.parametrize("regime", [0, 1, 2])
@pytest.mark.parametrize("d,nrhs", [(2, 1), (4, 17), (6, 1), (7, 5), (20, 16), (27, 32)])
def test_close_points(kind, regime, d, nrhs):
    ell = ELL[kind][regime]
    scale = np.sqrt(ell) if kind == "gaussian" else ell
    rng = np.random.default_rng(1000 * d + nrhs)
    b = W.dim_weights(d, 1.0)

    def partner(P):
        Q = P + 0.3 * scale / np.sqrt(d) * rng.standard_normal(P.shape)
        Q[:10] = P[:10]
        return Q

    A = W.points(150, d, 1.0, 5)
    X = np.concatenate([A, partner(A)])
    x = rng.standard_normal((300, nrhs))
    op = dw.fmm_create(dw.build_tree(torch.from_numpy(X).cuda(), b, 512, 0.8), kind, ell, 2, max_nrhs=nrhs)
    xd = torch.from_numpy(x).cuda()
    yd = torch.empty_like(xd)
    dw.fmm_matvec(op, xd, yd)
    errs = [(yd.cpu().numpy(), dense(kind, ell, X, X, x))]
    for m in (100, 300):  # one piece of targets, three
        T = partner(X[:m])
        zd = torch.empty((m, nrhs), dtype=torch.float64, device="cuda")
        dw.eval_apply(dw.eval_create(op, torch.from_numpy(T).cuda()), xd, zd)
        errs.append((zd.cpu().numpy(), dense(kind, ell, T, X, x)))
    errs = [np.linalg.norm(a - r) / np.linalg.norm(r) for a, r in errs]
    print(f"[close] {kind} ell={ell:g} d={d} nrhs={nrhs}: " + " ".join("%.1e" % e for e in errs), flush=True)
    if kind == "exponential":
        bound = 6e-15
    elif regime == 0:
        bound = 3e-13
    else:
        bound = 5e-15 if d <= 4 else 2.4e-14
    assert max(errs) <= bound
