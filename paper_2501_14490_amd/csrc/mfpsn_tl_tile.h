// Tile plan of the time-last kernels (mfpsn_tl_tile.hip): how a wave's 64
// lanes split the columns and time steps of a tile, and the order in which
// the tiles are walked.  Host code, shared with a CPU test.
//
// A tile is G consecutive columns over all T steps (nseg == 1), or one
// segment of `seg` steps of one column.  Lane = row * Q + q (Q = 64 / G):
// lane q of a row walks residue class q mod ncls of the dilation, and of the
// m chunks of that class (of equal length but the last) chunk q / ncls.
//
// Tiles come in groups with one set of channels, walked group by group, so a
// wave keeps its taps and its grad_w sums in registers over a whole group:
//   by_channel: group p is channel p; its tiles are (n, block of G columns of
//               the row of S, segment);
//   otherwise : group p is the columns p G .. of the S*C columns of a sample
//               (several channels per tile); its tiles are the samples n.
#pragma once

#include <stdint.h>

namespace mfpsn {

constexpr int kTileLdsMax = 65536;     // most LDS bytes of one wave's tile
constexpr int kTileMinSeg = 256;       // shortest segment of columns split for lack of them
constexpr int kTileMaxSpan = 1024;     // longest history (k-1) d of the segment tiles

struct TileGeom {
    int32_t T, C, S, d;     // d: at most T when the column is whole (the taps beyond reach nothing)
    int32_t G, Q, m, ncls;  // rows per tile, lanes per row, chunks per class, classes walked
    int32_t seg, nseg;      // steps per segment, segments per column
    int32_t span;           // history staged before (and, backward, after) a segment; 0: whole columns
    int32_t by_channel;
    int32_t sblk;           // by_channel: blocks of G columns per row of S
    int32_t CH;             // channels a tile can meet
    int32_t np;             // groups
    int32_t split;          // a channel may lie in two groups
    int32_t by_z;           // which numbering of the partial sums (tile_slot)
    int32_t Cp;             // slots of one wave that meets every group
    // Rows of an image whose bytes are a multiple of 16 get one word of padding
    // (G > 1), so that the lanes of different rows reading one step do not
    // meet in a few banks; a 16-byte piece then never spans rows.  Other rows
    // lie as in memory (an odd number of words, or of pairs of words).
    int32_t xs, os;         // elements from row to row of the images
    uint32_t tdiv;          // e / T = umulhi(e, tdiv) for e < 64 T
    int32_t lds_x, lds;     // LDS bytes before the second image, and in all
    int64_t Z, tiles;       // tiles per group, and in all
};

#ifdef __HIPCC__
#define MFPSN_TILE_FN __host__ __device__ inline
#else
#define MFPSN_TILE_FN inline
#endif

// Longest chunk of a class in a window of W steps.  Long chunks are odd: the
// lanes of a column then start in different banks (64, 4 bytes each) for
// the usual d = 1, 2, 4, for at most one step in 24 more.
MFPSN_TILE_FN int tile_chunk(const TileGeom& g, int W)
{
    const uint32_t d = (uint32_t)g.d, m = (uint32_t)g.m;
    const int R = (int)((((uint32_t)W + d - 1) / d + m - 1) / m);
    return R >= 24 ? R | 1 : R;
}

// Slot of the first of wave w's sums of group p, which it meets first at
// tile z of the group.  A wave walks consecutive tiles, so along the walk
// either the wave or the group goes up; channels of a group are numbered on
// from those before it (one more per group where groups split a channel), so
// no two (wave, group) pairs share a slot.  by_z numbers by the first tile
// instead of the wave: Z Cp slots whatever the number of waves.
MFPSN_TILE_FN int64_t tile_slot(const TileGeom& g, int64_t w, int64_t z, int p)
{
    const int64_t cum = g.by_channel ? p : (int64_t)p * g.G / g.S + (g.split ? p : 0);
    return (g.by_z ? z * g.Cp : w * g.CH) + cum;
}

// Waves per CU that the kernels' registers allow
inline int tile_waves_by_regs(bool backward, int k)
{
    return backward ? (k <= 8 ? 16 : k <= 16 ? 12 : 8) : (k <= 8 ? 24 : k <= 16 ? 20 : 12);
}

// Bytes of one wave's tile: the image of x (es bytes per element, 16-byte
// pieces as they lie in memory), then the second image (os bytes per
// element: 4 for dH or H, 1 for spikes), each with room for the walks' one
// step of read-ahead on either side.
inline void tile_lds(TileGeom& g, int es, int os, bool backward)
{
    g.xs = g.T + (g.G > 1 && (int64_t)g.T * es % 16 == 0 ? 4 / es : 0);
    g.os = g.T + (g.G > 1 && (int64_t)g.T * os % 16 == 0 ? 4 / os : 0);
    g.tdiv = g.T > 1 ? (uint32_t)(((uint64_t)1 << 32) / (uint64_t)g.T + 1) : 0;
    const int64_t ahead = backward ? g.span : 0;  // steps after a segment the backward needs
    const int64_t xn = g.nseg == 1 ? (int64_t)g.G * g.xs : (int64_t)g.seg + g.span + ahead;
    const int64_t on = g.nseg == 1 ? (int64_t)g.G * g.os : g.seg + ahead;
    const int64_t v = 16 / es;
    const int64_t xb = (xn + 2 * v + g.d) * es, ob = (on + 2 * v + 2 * (int64_t)g.d + 16) * os;
    const int64_t lx = (xb + g.d * os + 15) / 16 * 16;
    const int64_t all = (lx + ob + 15) / 16 * 16;
    g.lds_x = (int32_t)(lx < (1 << 30) ? lx : 1 << 30);
    g.lds = (int32_t)(all < (1 << 30) ? (all > 576 ? all : 576) : 1 << 30);
}

// Groups, slots and tiles of a plan whose G, nseg and by_channel are set
inline void tile_groups(TileGeom& g, int N, int64_t slots)
{
    const int64_t SC = (int64_t)g.S * g.C;
    if (g.by_channel) {
        g.sblk = (g.S + g.G - 1) / g.G;
        g.CH = 1;
        g.np = g.C;
        g.split = 0;
        g.Cp = g.C;
        g.Z = (int64_t)N * g.sblk * g.nseg;
    } else {
        g.sblk = 1;
        g.split = g.G % g.S != 0;
        g.CH = g.split ? (g.G + g.S - 2) / g.S + 1 : g.G / g.S;
        g.np = (int32_t)((SC + g.G - 1) / g.G);
        g.Cp = g.C + (g.split ? g.np - 1 : 0);
        g.Z = N;
    }
    g.tiles = (int64_t)g.np * g.Z;
    g.by_z = slots >= 0 && g.Z * g.Cp <= slots;
}

// Waves of a launch: at most `resident`, each taking ceil(tiles / waves)
// consecutive tiles, and (backward) at most as many as the slots of partial
// sums allow (slots < 0: no limit).  0: they do not even serve one wave.
inline int64_t tile_waves(const TileGeom& g, int64_t resident, int64_t slots)
{
    int64_t w = resident < g.tiles ? resident : g.tiles;
    if (slots >= 0 && !g.by_z) {
        const int64_t most = slots < g.Cp ? 0 : (slots - g.Cp) / g.CH + 1;
        w = w < most ? w : most;
    }
    return w;
}

// Whether the slots of partial sums keep a backward plan from the waves that
// fit (256 CUs; by registers and by LDS)
inline bool tile_short_of_waves(const TileGeom& g, int k, int64_t slots)
{
    const int64_t by_lds = 163840 / ((g.lds + 1279) / 1280 * 1280), by_regs = tile_waves_by_regs(true, k);
    const int64_t fit = 256 * (by_lds < by_regs ? by_lds : by_regs);
    return tile_waves(g, fit, slots) < tile_waves(g, fit, -1);
}

// The plan for one call (es: bytes of a stored element; slots: partial sums
// the backward's workspace holds, k + 1 values each; < 0: the forward, with its
// potentials kept if want_h).
// Returns false when no tile fits: histories above kTileMaxSpan of columns that
// are too long.  Whole columns up to 20 KB of LDS per tile (columns no longer
// than their history in any case), else segments.
//
// G is chosen by an estimate of the launch's time.  A tile costs R steps (the
// longest chunk), 0.7 of a step (forward 0.25) per history step of a cut class
// and 1.5 steps (forward 6) for the rest.  Fitted on MI355X: f32, T = 250,
// k = 16, d = 2, 131,072 columns, backward us at G = 1, 2, 4, 6, 8: 364, 290,
// 206, 181, 205; T = 32, k = 8, d = 1, 1 M columns at G = 8, 16, 32, 64: 213,
// 149, 116, 161.  The losses at the largest G come from LDS: below the waves
// per SIMD that the registers allow the time grows as their inverse.  One
// wave alone on a SIMD takes about twice its instructions' issue time, and
// 1024 SIMDs share the tiles: few columns take the G that spreads them.
inline bool tile_plan(TileGeom& g, int T, int N, int C, int S, int k, int dilation, int es, int64_t slots,
                      bool want_h = false)
{
    const bool backward = slots >= 0;
    const int os = backward || want_h ? 4 : 1;
    const int64_t span = (int64_t)(k - 1) * dilation;
    const double halo = (backward ? 0.7 : 0.25) * (k - 1), fixed = backward ? 1.5 : 6.0;
    const int by_regs = tile_waves_by_regs(backward, k);
    g.T = T;
    g.C = C;
    g.S = S;
    g.nseg = 1;
    g.seg = T;
    g.span = 0;
    g.d = k == 1 ? 1 : (dilation < T ? dilation : T);
    g.ncls = g.d < T ? g.d : T;
    double best = 0.0;
    TileGeom out = g;
    bool found = false;
    const int L = (int)(((int64_t)T + g.d - 1) / g.d);
    for (int G = 1; G <= 64 && (G == 1 || G * (int64_t)g.ncls <= 64); ++G) {
        TileGeom t = g;
        t.G = G;
        t.Q = 64 / G;
        t.m = t.Q / t.ncls > 0 ? t.Q / t.ncls : 1;
        t.m = t.m < L ? t.m : L;
        t.by_channel = G <= S;
        tile_lds(t, es, os, backward);
        if (t.lds > 20480 || (!t.by_channel && G > (int64_t)S * C))
            break;
        tile_groups(t, N, slots);
        const int64_t waves = tile_waves(t, 3072, slots);
        if (waves < 1)
            continue;
        const int passes = (t.ncls + t.Q - 1) / t.Q;
        const double tile = passes * (tile_chunk(t, T) + (t.m > 1 ? halo : 0.0)) + fixed;
        const double by_lds = 163840.0 / t.lds, starved = by_lds < by_regs ? by_regs / by_lds : 1.0;
        const double alone = 2.0 * tile * (double)((t.tiles + waves - 1) / waves);
        const double all = tile * (double)t.tiles / 1024 * starved;
        const double cost = alone > all ? alone : all;
        if (!found || cost < best) {
            best = cost;
            out = t;
            found = true;
        }
    }
    // few long columns: segments down to kTileMinSeg steps, so that one wave per
    // SIMD has work (not more than the backward's slots allow waves).  64 columns
    // of 2000 steps, f32 k = 8, forward and backward us: two segments 8.0, 22.7,
    // seven 5.5, 13.7; from 960 columns on the longer segments win (k = 32, T =
    // 700: backward 29.9 us whole, 37.6 in two).
    const int64_t M = (int64_t)N * C * S, least = span > kTileMinSeg ? span : kTileMinSeg;
    int64_t few = M <= 512 ? (1024 + M - 1) / M : 1;
    if (slots >= 0 && few > (slots - C + 1) / M)
        few = (slots - C + 1) / M;
    if (few > T / least)
        few = T / least;
    if (span > kTileMaxSpan)
        few = 1;
    if (!found || few > 1) {
        // segments of one column: at least as long as the history, and long
        // enough that the history computed twice (backward) is a small share
        if (span > kTileMaxSpan || T < 2)
            return false;
        if (!found && span >= T) {
            // a column no longer than its history makes one segment: whole, in
            // a larger tile (at most 24 T bytes, T <= 1024)
            g.G = 1;
            g.Q = 64;
            g.m = 64 / g.ncls > 0 ? 64 / g.ncls : 1;
            g.m = g.m < L ? g.m : L;
            g.by_channel = 1;
            tile_lds(g, es, os, backward);
            tile_groups(g, N, slots);
            return g.lds <= kTileLdsMax && tile_waves(g, 1, slots) > 0;
        }
        g.d = k == 1 ? 1 : dilation;
        g.ncls = g.d < T ? g.d : T;
        g.G = 1;
        g.Q = 64;
        g.m = 64 / g.ncls > 0 ? 64 / g.ncls : 1;
        g.by_channel = 1;
        g.span = (int32_t)span;
        const int64_t top = span > 512 || backward ? 2048 : 1024;
        int64_t n = (T + top - 1) / top;
        n = n > 2 ? n : 2;
        n = n > few ? n : few;
        g.seg = (int32_t)((T + n - 1) / n);
        if (g.seg < span)
            g.seg = (int32_t)span;
        g.nseg = (T + g.seg - 1) / g.seg;
        tile_lds(g, es, os, backward);
        tile_groups(g, N, slots);
        if (g.nseg == 1 || g.lds > kTileLdsMax || tile_waves(g, 1, slots) < 1)
            return false;
        out = g;
    }
    g = out;
    return true;
}

}  // namespace mfpsn
