"""The table form of 2^t in the FP64 nearfield kernels, replayed on the CPU.

2^t = 2^(n / 1024) (1 + (2^f - 1)) with n the low word of t + 1.5 2^42, |f| <= 2^-11: the table (built
by the compiler in 126-bit fixed point, the steps replayed here in integers) is correctly rounded, the
cubic is the generator's, and the whole sequence, every fused multiply-add rounded once, stays within
half an ulp (table) + half an ulp (last operation) + 9.4e-17 (cubic) = 3.2e-16, and a little for the
cubic's own rounding.
"""
import importlib.util
import io
import pathlib
import re
from contextlib import redirect_stdout
from fractions import Fraction

import numpy as np

CSRC = pathlib.Path(__file__).resolve().parents[1] / "paper_2402_09531_amd" / "csrc"
SRC = (CSRC / "kernels.hip").read_text()
BOUND = 3.4e-16


def fma(a, b, c):
    return np.array([float(Fraction(x) * Fraction(y) + Fraction(z)) for x, y, z in np.broadcast(a, b, c)])


def table():
    s1, s0 = (int(v, 16) for v in re.search(r"s1 = (0x[0-9a-f]+), s0 = (0x[0-9a-f]+);", SRC).groups())
    m64 = (1 << 64) - 1
    x, out = 1 << 126, []
    for j in range(1024):
        m = (x + (1 << 73)) >> 74
        out.append(((1022 << 52) + m - (j << 42)) & m64)
        x1, x0 = x >> 64, x & m64
        mid = x1 * s0 + x0 * s1 + ((x0 * s0) >> 64)
        assert mid < 1 << 128
        x = ((x1 * s1) << 2) + (mid >> 62)
    return np.array(out, dtype=np.uint64)


def cubic():
    body = SRC[SRC.index("double exp2m1_short(double f)"):]
    body = body[:body.index("\n}\n")]
    return [float(re.search(r"double p = ([0-9.e+-]+);", body).group(1))] + \
        [float(v) for v in re.findall(r"fma\(p, f, ([0-9.e+-]+)\)", body)]


def exp2_tab(t, tab, c):
    big = 6597069766656.0
    assert big == 1.5 * 2.0 ** 42
    m = t + big
    f = t - (m - big)
    assert np.all(np.abs(f) <= 2.0 ** -11)
    p = fma(fma(np.full_like(f, c[0]), f, c[1]), f, c[2]) * f
    n = (m.view(np.int64) & 0xFFFFFFFF).astype(np.uint32).view(np.int32).astype(np.int64)
    w = tab[n & 1023]
    hi = ((w >> np.uint64(32)).astype(np.int64) + (n << 10)) & 0xFFFFFFFF   # 32-bit add to the high word
    v = ((hi.astype(np.uint64) << np.uint64(32)) | (w & np.uint64(0xFFFFFFFF))).view(np.float64)
    return fma(v, p, v)


def test_table_is_correctly_rounded():
    tab = table()
    prec = 200
    import math
    root = 2 << prec
    for _ in range(10):
        root = math.isqrt(root << prec)
    x = 1 << prec
    for j in range(1024):
        want = float(Fraction(x, 1 << prec))
        got = np.array([(int(tab[j]) + (j << 42)) & ((1 << 64) - 1)], dtype=np.uint64).view(np.float64)[0]
        assert got == want, j
        x = (x * root) >> prec


def test_cubic_matches_generator():
    spec = importlib.util.spec_from_file_location("gen_exp_coeffs", CSRC / "gen_exp_coeffs.py")
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    buf = io.StringIO()
    with redirect_stdout(buf):
        mod.main()
    gen = [float(v) for v in re.findall(r"d\d = np\.float64\(([0-9.e+-]+)\)", buf.getvalue())]
    assert cubic() == gen[::-1] and len(gen) == 3


def test_relative_error():
    tab, c = table(), cubic()
    rng = np.random.default_rng(5)
    t = np.concatenate([rng.uniform(-2.0, 2.0, 20_000), rng.uniform(-1020.0, 1020.0, 20_000),
                        (np.arange(-300, 300) + 0.5) / 1024, [-1020.0, 1020.0, 0.0, 1e-300]])
    ref = np.exp2(t.astype(np.longdouble))
    rel = np.abs((exp2_tab(t, tab, c) - ref) / ref).astype(np.float64)
    assert rel.max() <= BOUND, rel.max()
    assert np.array_equal(exp2_tab(np.arange(-1020.0, 1021.0), tab, c), np.exp2(np.arange(-1020.0, 1021.0)))
