"""The tile plan of the time-last kernels (csrc/mfpsn_tl_tile.h) on the CPU: the
host header is compiled with g++ and a driver walks the plan of many calls
as the kernels do.

Checked for every call: each (column, step) is computed by exactly one lane of
one tile; every LDS element a walk touches (history, read-ahead, staged
16-byte pieces at any alignment) lies inside its image; no two (wave, group)
pairs share a slot of partial sums and every slot fits the workspace.
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
#include <cstdlib>
#include <algorithm>
#include <set>
#include <vector>
#include "mfpsn_tl.h"
using namespace mfpsn;
#define CHECK(x) do { if (!(x)) { printf("line %d: %s\n", __LINE__, #x); return 1; } } while (0)
// bwd 0: forward, 1: backward, 2: forward that keeps H
int one(int T, int N, int C, int S, int k, int d, int es, int kind, long resident)
{
    const bool bwd = kind == 1;
    const long M = (long)N * C * S, span = (long)(k - 1) * d;
    const long slots = bwd ? tl_bwd_slots(M, T, C, N, span) : -1;
    TileGeom g;
    if (!tile_plan(g, T, N, C, S, k, d, es, slots, kind == 2)) {
        CHECK(T > 64 && span > kTileMaxSpan);  // what the entry points refuse, or run untiled
        return 0;
    }
    CHECK(g.lds <= 65536 && g.lds_x < g.lds && g.lds_x % 16 == 0 && g.G * g.Q <= 64 && g.G >= 1);
    const long waves = tile_waves(g, resident, slots);
    CHECK(waves >= 1);
    if (M <= 512 && !bwd && T >= 512 && span <= 256)  // few long columns are cut, for more waves
        CHECK(g.nseg >= std::min(T / 256, (int)(1024 / M)));
    const long chunk = (g.tiles + waves - 1) / waves;
    const int os = kind > 0 ? 4 : 1, v = 16 / es;
    std::vector<unsigned char> seen(M * T, 0);
    std::set<long> used;
    for (long w = 0; w * chunk < g.tiles; ++w) {
        int cur = -1;
        for (long t = w * chunk; t < std::min((w + 1) * chunk, (long)g.tiles); ++t) {
            const int p = (int)(t / g.Z);
            const long z = t - p * g.Z;
            long col0; int rows, t0 = 0;
            if (g.by_channel) {
                const long per = (long)g.sblk * g.nseg, n = z / per, rest = z % per;
                col0 = (n * C + p) * S + rest / g.nseg * g.G;
                rows = std::min(g.G, S - (int)(rest / g.nseg) * g.G);
                t0 = (int)(rest % g.nseg) * g.seg;
            } else {
                col0 = z * (long)S * C + (long)p * g.G;
                rows = (int)std::min((long)g.G, (long)S * C - (long)p * g.G);
            }
            CHECK(rows >= 1 && t0 < T);
            if (p != cur) {
                cur = p;
                if (bwd) {  // the slots of this wave's sums of group p
                    const long s0 = tile_slot(g, w, z, p);
                    const int c0 = g.by_channel ? p : (int)((long)p * g.G / S);
                    const int c1 = g.by_channel ? p : (int)(((long)p * g.G + rows - 1) / S);
                    CHECK(c1 - c0 < g.CH);
                    for (int c = c0; c <= c1; ++c) {
                        CHECK(s0 + c - c0 < slots);
                        CHECK(used.insert(s0 + c - c0).second);
                    }
                    // and where the reduction looks for them
                    const long zf = w * chunk - p * g.Z;
                    CHECK(tile_slot(g, w, zf > 0 ? zf : 0, p) == s0);
                }
            }
            const int own = std::min(g.seg, T - t0), win = bwd ? std::min(own + g.span, T - t0) : own;
            const int before = std::min(g.span, t0);
            const long count = g.nseg == 1 ? (long)rows * T : win;
            CHECK(t0 == 0 || before >= span);
            const bool xpad = g.xs != T, opad = g.os != T;
            CHECK(!xpad || (g.G > 1 && T * es % 16 == 0 && (g.xs - T) * es == 4));
            CHECK(!opad || (g.G > 1 && T * os % 16 == 0 && (g.os - T) * os == 4));
            CHECK(xpad || g.G == 1 || T * es % 16 != 0);
            for (long e = 0; T > 1 && e < count; ++e)  // rows by the multiplied reciprocal
                CHECK((long)(((unsigned long)e * g.tdiv) >> 32) == e / T || !(xpad || opad));
            for (int off = 0; off < v; ++off) {
                CHECK(((off + before + count + v - 1) / v * v + (rows - 1) * (g.xs - T)) * es <= g.lds_x);
                CHECK(g.lds_x + ((off + count + v - 1) / v * v + (rows - 1) * (g.os - T)) * os <= g.lds);
            }
            if (!bwd)
                CHECK(g.lds_x + (16 + count + (rows - 1) * (g.os - T)) * os <= g.lds);
            for (int lane = 0; lane < 64; ++lane) {
                const int row = std::min(lane / g.Q, g.G - 1), q = lane - row * g.Q;
                if (!(q < g.ncls * g.m && lane < g.G * g.Q) || row >= rows)
                    continue;
                const int ch = q / g.ncls;
                for (int r = q - ch * g.ncls; r < g.ncls; r += g.ncls > 64 ? 64 : g.ncls)
                    for (int pass = 0; pass < 2; ++pass) {
                        const int W = pass == 0 ? win : own;
                        const int L = r < W ? (W - r + g.d - 1) / g.d : 0;
                        const int top = tile_chunk(g, W);
                        const int j0 = std::min(ch * top, L), j1 = std::min(j0 + top, L);
                        // read-ahead, unconditional reads and history
                        const long lo = (long)row * g.xs + r + (long)j0 * g.d, hi = (long)row * g.xs + r + (long)j1 * g.d;
                        const long dlo = lo + row * (g.os - g.xs), dhi = hi + row * (g.os - g.xs);
                        if (pass == 0) {
                            const int hist = t0 > 0 ? k : j0;
                            for (int b = 1; b < k; ++b)
                                if (b <= hist && (g.m > 1 || t0 > 0))
                                    CHECK(before + lo - (long)b * g.d >= 0);
                            CHECK((v - 1 + before + std::max(hi, lo) + 1) * es <= g.lds_x);
                            CHECK(g.lds_x + (v - 1 + std::max(dhi, dlo) + 1) * os <= g.lds);
                        } else {
                            const int Lw = r < win ? (win - r + g.d - 1) / g.d : 0;
                            CHECK(g.m > 1 || g.nseg > 1 || Lw == j1);  // nothing after the chunk to read
                            for (int b = 1; b < k; ++b)
                                if (b <= Lw - j1)
                                    CHECK(dhi - g.d + (long)b * g.d < (long)row * g.os + (g.nseg == 1 ? T : win));
                            CHECK(g.lds_x + (dlo - g.d) * os >= 0);
                            for (int j = j0; j < j1; ++j) {
                                const long e = (col0 + row) * T + t0 + r + (long)j * g.d;
                                CHECK(e < M * T && !seen[e]);
                                seen[e] = 1;
                            }
                        }
                    }
            }
        }
    }
    for (unsigned char s : seen)
        CHECK(s);
    return 0;
}
int main()
{
    int T, N, C, S, k, d, es, bwd;
    long resident;
    while (scanf("%d %d %d %d %d %d %d %d %ld", &T, &N, &C, &S, &k, &d, &es, &bwd, &resident) == 9)
        if (one(T, N, C, S, k, d, es, bwd, resident)) {
            printf("T %d N %d C %d S %d k %d d %d es %d bwd %d resident %ld\n", T, N, C, S, k, d, es, bwd, resident);
            return 1;
        }
    return 0;
}
"""

EDGES = [(1, 1, 1, 1, 1, 1), (2, 1, 3, 1, 2, 5), (64, 1, 100, 1, 8, 1), (64, 1, 1000, 3, 4, 3), (65, 2, 5, 7, 3, 70),
         (250, 3, 70, 1, 16, 4), (30, 1, 3, 1936, 8, 3), (48, 1, 1000, 3, 2, 3), (1300, 1, 2, 1, 32, 8),
         (2049, 1, 2, 1, 32, 33), (4096, 1, 3, 1, 2, 1024), (5000, 1, 1, 2, 33 - 1, 33), (300, 1, 2, 2, 1, 500),
         (2100, 1, 1, 2, 3, 512), (1500, 2, 1, 3, 2, 1400), (100, 2, 3, 5, 2, 99),
         (900, 2, 3, 1, 2, 1000), (1020, 1, 2, 1, 2, 1024), (2000, 4, 4, 1, 8, 1), (700, 1, 3, 5, 16, 16)]


@pytest.fixture(scope="module")
def walk(tmp_path_factory):
    """Runs the driver over calls (T, N, C, S, k, d, es, 0 forward / 1 backward / 2 forward that
    keeps H, resident waves); returns what it found wrong."""
    path = tmp_path_factory.mktemp("tile_plan")
    src, exe = path / "drv.cpp", path / "drv"
    src.write_text(DRIVER)
    subprocess.run(["g++", "-std=c++20", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include", f"-I{CSRC}",
                    str(src), "-o", str(exe)], check=True, capture_output=True)

    def run(calls):
        lines = "\n".join(" ".join(map(str, c)) for c in calls)
        out = subprocess.run([str(exe)], input=lines, capture_output=True, text=True)
        return "" if out.returncode == 0 else out.stdout or f"exit {out.returncode}"

    return run


@pytest.mark.parametrize("seed", [0, 1, 2])
def test_every_step_has_one_lane_and_every_access_its_room(walk, seed):
    rng = random.Random(seed)
    calls = list(EDGES) if seed == 0 else []
    while len(calls) < 400:
        T = int(2 ** rng.uniform(0, 12.5))
        S, C, N = (int(2 ** rng.uniform(0, m)) for m in (7, 6, 3))
        if T * S * C * N <= 300_000:
            calls.append((T, N, C, S, rng.randint(1, 32), int(2 ** rng.uniform(0, rng.choice([3, 11])))))
    assert walk((*c, es, bwd, resident) for c in calls for es in (2, 4) for bwd in (0, 1, 2)
                for resident in (1, 7, 4096)) == ""


def test_histories_about_as_long_as_the_column_have_a_plan(walk):
    """Every T from 65 to 1100 with dilations at and beyond it, up to the longest history: columns too long for
    20 KB whole and no longer than their history (order 2: f32 from T = 849, 16-bit from T = 1017)."""
    assert walk((T, 1, 2, 1, k, d, es, bwd, 7) for T in range(65, 1101) for k in (2, 3)
                for d in {T - 1, T, T + 1, 1024 // (k - 1) - 1, 1024 // (k - 1)} if d * (k - 1) <= 1024
                for es in (2, 4) for bwd in (0, 1)) == ""
