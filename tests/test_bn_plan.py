"""The walk plan of the batch-normalization backward (csrc/mfpsn_bn.h) on the
CPU: chunks cover every class, a thread's items lie in one channel, and the
plan needs no more workspace than the shared plan that sizes it; orders outside
15 to 22 keep the shared plan; the audio layer's whole classes fill two waves
per SIMD with two items each.
"""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2501_14490_amd", "csrc")

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")

DRIVER = r"""
#include <cstdio>
#include "mfpsn_bn.h"
using namespace mfpsn;
#define CHECK(x) do { if (!(x)) { printf("T %d N %d C %d S %d k %d d %d: %s\n", T, N, C, S, k, d, #x); return 1; } } while (0)
int main()
{
    for (int T : {1, 7, 30, 64, 250, 1000, 4096}) for (int N : {1, 3, 17, 256}) for (int C : {1, 100, 512})
    for (int S : {1, 35}) for (int k : {1, 8, 14, 15, 16, 22, 23, 32}) for (int d : {1, 2, 4, 5000}) {
        BnGeom g{};
        g.T = T; g.N = N; g.C = C; g.S = S; g.k = k; g.d = d;
        g.M = (size_t)N * C * S; g.tq = T / d; g.tr = T % d;
        bn_plan(g);
        BnGeom b = g;
        bn_backward_plan(b);
        if (k < 15 || k > 22)
            CHECK(b.G == g.G && b.lc == g.lc && b.nch == g.nch);
        const int L = (T + d - 1) / d;
        CHECK(b.lc >= 1 && (int64_t)b.lc * b.nch >= L && (int64_t)b.lc * (b.nch - 1) < L);
        CHECK(b.items == (size_t)b.nch * d * b.M);
        CHECK(b.G % kBnThreads == 0 && b.G >= 1);
        CHECK(b.G >= b.items || b.G % ((size_t)S * C) == 0);
        CHECK(b.G <= g.G && b.NG <= g.NG && b.R == (int32_t)((b.G + (size_t)S * C - 1) / ((size_t)S * C)));
        CHECK(b.NG == (b.R + kBnRowGroup - 1) / kBnRowGroup);
        if (T == 250 && N == 256 && C == 512 && S == 1 && k == 16 && d == 2)
            CHECK(b.nch == 1 && b.G == 131072 && b.items == 2 * b.G);
    }
    return 0;
}
"""


def test_backward_plan(tmp_path):
    src, exe = tmp_path / "plan.cpp", tmp_path / "plan"
    src.write_text(DRIVER)
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", f"-I{CSRC}",
                    f"-I{os.path.join(ROOT, 'include')}", str(src), "-o", str(exe)], check=True)
    p = subprocess.run([str(exe)], capture_output=True, text=True)
    assert p.returncode == 0, p.stdout


SLOWER = r"""
#include "mfpsn_bn.h"
using namespace mfpsn;
int main()
{
    for (int k : {15, 16}) {
        BnGeom g{};
        g.T = 128; g.N = 64; g.C = 100; g.S = 13; g.k = k; g.d = 2;
        g.M = (size_t)g.N * g.C * g.S;
        bn_plan(g);
        BnGeom b = g;
        bn_backward_plan(b);
        if (b.G != g.G || b.nch != g.nch)
            return 1;
    }
    return 0;
}
"""


def test_a_plan_hardly_better_by_its_estimate_is_not_taken(tmp_path):
    """[128,64,100,13] d = 2: half the waves, one chunk instead of two; 70.4 us instead of 67.3 at order 16."""
    src, exe = tmp_path / "slower.cpp", tmp_path / "slower"
    src.write_text(SLOWER)
    subprocess.run(["g++", "-std=c++17", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", f"-I{CSRC}",
                    f"-I{os.path.join(ROOT, 'include')}", str(src), "-o", str(exe)], check=True)
    assert subprocess.run([str(exe)]).returncode == 0
