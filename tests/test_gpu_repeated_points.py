"""Repeated points under the exponential kernel: its square root makes 1e-8 of a rounding of r^2, so the
distance of a point to its copy has to come out as zero.

64 points and their copies in one leaf, the length scale a fiftieth of the smallest distance (a value of
2e-22 there, and a thousandth of it for the clamped kernel): the row sums for x = 1 are 1 + 1 exactly.
The nearfields of one rhs (with and without the norms in the Gram operands: d mod 4 in {1, 2} and not)
and of several, leaves above 128 points and evaluation at the points themselves, and a batch.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import paper_2402_09531_amd as dw  # noqa: E402
from paper_2402_09531_amd import workloads as W  # noqa: E402


@pytest.mark.parametrize("shrink", [50.0, 5e4])
@pytest.mark.parametrize("d", [3, 4, 6, 8, 9, 16, 20, 23, 28])
def test_exponential(d, shrink):
    A = W.points(64, d, 0.0, 5)
    dist = np.sqrt(((A[:, None] - A[None]) ** 2).sum(-1)) + 1e3 * np.eye(64)
    ell = float(dist.min() / shrink)
    b = W.dim_weights(d, 0.0)
    Xd = torch.from_numpy(np.concatenate([A, A])).cuda()
    print(f"[repeated] d={d} ell={ell:g}", flush=True)
    for nrhs in (1, 5):
        op = dw.fmm_create(dw.build_tree(Xd, b, 128, 0.8), "exponential", ell, 1, max_nrhs=nrhs)
        x = torch.ones((128, nrhs), dtype=torch.float64, device="cuda")
        y = torch.empty_like(x)
        dw.fmm_matvec(op, x, y)
        assert bool((y == 2).all())
        dw.eval_apply(dw.eval_create(op, Xd), x, y)
        assert bool((y == 2).all())
        if nrhs == 1:
            dw.batch_matvec(dw.batch_create([op]), [x], [y])
            assert bool((y == 2).all())
    big = dw.fmm_create(dw.build_tree(torch.cat([Xd, Xd]), b, 256, 0.8), "exponential", ell, 1)
    x = torch.ones((256, 1), dtype=torch.float64, device="cuda")
    y = torch.empty_like(x)
    dw.fmm_matvec(big, x, y)
    assert bool((y == 4).all())
