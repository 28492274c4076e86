"""The first solves of a process allocate no memory that the GPU can see.

Counted in a process of its own, as the mappings of the GPU's device file before and after the first solve
of a small operator (and after a second operator's), once the runtime's own buffers are there: another
operator has been solved with a progress callback (which reads the state by ordinary copies) and torch has
copied into pinned memory.
"""
import pathlib
import subprocess
import sys

import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

CHILD = """
import numpy as np, torch
import paper_2402_09531_amd as dw
from paper_2402_09531_amd import workloads as W

X, b = W.points(1024, 4, 2.0, 7), W.dim_weights(4, 2.0)
Xd = torch.from_numpy(X).cuda()
f = torch.from_numpy(np.sin(X.sum(axis=1))[:, None].copy()).cuda()

def op(**kw):
    return dw.fmm_create(dw.build_tree(Xd, b, 64, 0.8), "matern32", 1.0, 4, **kw)

def solve(o):
    a = torch.zeros_like(f)
    assert dw.fmm_solve(o, 1.0, f, a, 1e-8, 400)[0]["status"] == 0
    return a

def mapped():
    return sorted(l.split()[0] for l in open("/proc/self/maps") if "renderD" in l)

warm, first, second = op(progress=lambda it, rr: None), op(), op()
pinned, ev = torch.empty(16, dtype=torch.float64, pin_memory=True), torch.cuda.Event()
for _ in range(3):
    a = solve(warm)
    pinned.copy_(a[:16, 0], non_blocking=True)
    ev.record()
    ev.synchronize()
assert torch.equal(a, solve(warm))
before = mapped()
assert before
for o in (first, second):
    got = solve(o)
    after = mapped()
    assert after == before, [m for m in after if m not in before]
    assert torch.equal(got, a)
print("no new mapping")
"""


def test_first_solve_allocates_nothing():
    root = pathlib.Path(__file__).resolve().parents[1]
    got = subprocess.run([sys.executable, "-c", CHILD], cwd=root, capture_output=True, text=True, timeout=100)
    print(got.stdout, got.stderr[-2000:], flush=True)
    assert got.returncode == 0 and "no new mapping" in got.stdout
