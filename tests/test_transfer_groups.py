"""The launch groups of M2M and L2L, on the CPU: every level of the tree runs exactly once and in order, and
forming them allocates nothing (a matvec forms them on each call, under capture too, and is documented to
allocate nothing)."""
import pathlib
import subprocess

import pytest

CSRC = pathlib.Path(__file__).resolve().parents[1] / "paper_2402_09531_amd" / "csrc"
CLANG = pathlib.Path("/opt/rocm/llvm/bin/clang++")

MAIN = """
#include "device.hpp"
#include <cstdio>
#include <cstdlib>
#include <new>
static long allocs = 0;
void *operator new(size_t n) { ++allocs; return std::malloc(n ? n : 1); }
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, size_t) noexcept { std::free(p); }
int main()
{
    for (int up = 0; up < 2; ++up)
        for (int nx : {1, 11, 16, 33, 97, 128})
            for (int nrhs : {1, 2, 16, 32})
                for (int lo = 0; lo < 32; ++lo)
                    for (int hi = lo - 1; hi < 32; ++hi) {
                        const long before = allocs;
                        int next = up ? hi : lo, ok = 1;
                        for (const auto &g : dwfmm::xfer_groups(up, nx, nrhs, lo, hi)) {
                            // a group takes the levels root ... root + depth - 1, M2M the deepest first
                            ok &= g.depth >= 1 && (up ? g.root + g.depth - 1 : g.root) == next;
                            next = up ? g.root - 1 : g.root + g.depth;
                        }
                        ok &= next == (up ? lo - 1 : hi + 1) && allocs == before;
                        if (!ok) std::printf("up %d nx %d nrhs %d levels %d %d allocs %ld\\n", up, nx, nrhs, lo, hi, allocs - before);
                        if (!ok) return 1;
                    }
    std::printf("ok\\n");
}
"""


@pytest.mark.skipif(not CLANG.exists(), reason="no clang++")
def test_groups_cover_levels_without_allocation(tmp_path):
    src, exe = tmp_path / "groups.cpp", tmp_path / "groups"
    src.write_text(MAIN)
    subprocess.run([str(CLANG), "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", f"-I{CSRC}",
                    str(src), "-o", str(exe)], check=True)
    out = subprocess.run([str(exe)], capture_output=True, text=True)
    print(out.stdout)
    assert out.returncode == 0 and out.stdout.strip() == "ok"
