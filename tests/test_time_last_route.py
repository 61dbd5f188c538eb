"""Which kernels a time-last call on short columns goes to (csrc/mfpsn_tl.h) on
the CPU: the host headers are compiled with g++.

The calls below are measured ones (both kernels, MI355X) in which the other
choice is at least a tenth slower.  For calls of all kinds the slots of partial
sums of the column kernels (block + row of S columns) lie in the workspace.
"""
import os
import random
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2501_14490_amd", "csrc")

pytestmark = pytest.mark.skipif(shutil.which("g++") is None, reason="needs g++")

DRIVER = r"""
#include <cstdio>
#include "mfpsn_tl.h"
using namespace mfpsn;
int main()
{
    int T, N, C, S, k, d, dt;
    while (scanf("%d %d %d %d %d %d %d", &T, &N, &C, &S, &k, &d, &dt) == 7) {
        const long M = (long)N * C * S, slots = tl_bwd_slots(M, T, C, N, (long)(k - 1) * d);
        bool bwd = tl_by_columns(true, dt, M, T, k, d);
        TileGeom g;
        if (!bwd && tile_plan(g, T, N, C, S, k, d, dt == 0 ? 4 : 2, slots) && !tl_bears_few_waves(dt, T, k, d))
            bwd = tile_short_of_waves(g, k, slots);
        printf("%d %d %d\n", tl_by_columns(false, dt, M, T, k, d), bwd,
               !bwd || (M + 63) / 64 - 1 + ((long)N * C - 1) < slots);
    }
}
"""
DTYPE = {"f32": 0, "bf16": 1, "q8_8": 2}


@pytest.fixture(scope="module")
def routes(tmp_path_factory):
    """(forward by columns, backward by columns, its slots fit) of calls (T, N, C, S, k, d, dtype)."""
    path = tmp_path_factory.mktemp("route")
    src, exe = path / "drv.cpp", path / "drv"
    src.write_text(DRIVER)
    subprocess.run(["g++", "-std=c++20", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", f"-I{CSRC}",
                    str(src), "-o", str(exe)], check=True, capture_output=True)

    def run(calls):
        lines = "\n".join(" ".join(str(DTYPE.get(v, v)) for v in c) for c in calls)
        out = subprocess.run([str(exe)], input=lines, capture_output=True, text=True, check=True).stdout
        return [tuple(bool(int(v)) for v in line.split()) for line in out.splitlines()]

    return run


@pytest.mark.parametrize("call,fwd,bwd", [
    # columns / tiles, us, forward and backward: 21, 28 and 68, 77
    ((30, 16, 64, 546, 8, 3, "bf16"), True, True),
    ((16, 64, 128, 256, 4, 3, "bf16"), True, True),      # 153 / 273 together
    ((8, 16, 64, 2048, 4, 4, "f32"), True, True),        # 2.7 and 2.4 times
    ((24, 16, 64, 682, 4, 32, "q8_8"), True, True),      # 4.7 and 3.7 times
    ((64, 16, 64, 256, 8, 32, "bf16"), True, True),      # 1.9 and 1.6 times
    ((64, 16, 64, 256, 8, 1, "bf16"), False, False),     # 30, 21 and 93, 69
    ((32, 16, 64, 512, 8, 1, "f32"), None, False),       # 90, 68
    ((40, 16, 64, 409, 4, 2, "q8_8"), None, False),      # 1.6 times
    ((64, 16, 64, 256, 16, 2, "f32"), False, False),     # 44, 28 and 171, 95
    ((64, 1, 512, 1, 16, 1, "f32"), None, False),        # fewer columns yet: 39, 17
    ((40, 16, 64, 6, 16, 3, "f32"), None, True),         # few columns: 31, 38
    ((30, 16, 64, 546, 16, 2, "bf16"), None, False),     # many of a high order: 112, 78
    ((64, 16, 64, 30, 8, 4, "f32"), None, False),        # fewer waves than fit, and still faster
    ((64, 16, 64, 30, 8, 4, "bf16"), None, True),        # and not
    ((65, 16, 64, 252, 8, 33, "bf16"), False, False),    # no columns above 64 steps
])
def test_measured_calls_go_to_the_faster_kernels(routes, call, fwd, bwd):
    got_fwd, got_bwd, fits = routes([call])[0]
    assert got_bwd is bwd and fits
    assert fwd is None or got_fwd is fwd


def test_the_column_slots_lie_in_the_workspace(routes):
    rng = random.Random(0)
    calls = [(rng.randint(1, 64), *(int(2 ** rng.uniform(0, m)) for m in (8, 8, 10)), rng.randint(1, 32),
              int(2 ** rng.uniform(0, 7)), rng.choice(list(DTYPE))) for _ in range(2000)]
    assert all(fits for _, _, fits in routes(calls))
