// Internal interface of the batch-normalization kernels (mfpsn_bn.hip) for
// the C-ABI layer.  Not installed; not part of the ABI.
#pragma once

#include <hip/hip_runtime_api.h>
#include <stddef.h>
#include <stdint.h>

namespace mfpsn {

struct BnGeom {
    int32_t T, N, C, S, k, d;
    size_t M;        // N*C*S
    int32_t tq, tr;  // T = tq * d + tr: class r has tq + (r < tr) steps
    int32_t lc;      // class steps per walk chunk
    int32_t nch;     // chunks per class, ceil(ceil(T/d) / lc)
    size_t items;    // walk items, nch * d * M
    size_t G;        // walk threads: thread t takes items t, t + G, ...; all of
                     // them in channel ((t mod S*C) / S) (G is a multiple of
                     // S*C and of the block size, or no thread has two items)
    int32_t R;       // partial rows, ceil(G / (S*C)): thread t = row * S*C + j
    int32_t NG;      // row groups of the first reduction level, ceil(R / kBnRowGroup)
};
constexpr int kBnThreads = 256;
constexpr int kBnRowGroup = 16;

// Threads of a plan whose items are set: at most `most` (the items spread
// evenly, every thread in one channel), or one item per thread
inline void bn_threads(BnGeom& g, int64_t most)
{
    const int64_t SC = (int64_t)g.S * g.C, items = (int64_t)g.items;
    int64_t a = SC, b = kBnThreads;  // base = lcm(SC, block size)
    while (b != 0) {
        const int64_t t = a % b;
        a = b;
        b = t;
    }
    const int64_t base = SC > 0 ? SC / a * kBnThreads : kBnThreads;
    int64_t G;
    if (items == 0)
        G = kBnThreads;
    else if (base > items)
        G = (items + kBnThreads - 1) / kBnThreads * kBnThreads;  // one item per thread
    else {
        const int64_t per = (items + most - 1) / most;  // items per thread
        G = ((items + per - 1) / per + base - 1) / base * base;
    }
    g.G = (size_t)G;
    g.R = SC > 0 ? (int32_t)((G + SC - 1) / SC) : 1;
    g.NG = (g.R + kBnRowGroup - 1) / kBnRowGroup;
}

// Chunks of each class, nch as wished (rounded to chunks of one length)
inline void bn_chunks(BnGeom& g, int64_t nch)
{
    const int64_t L = ((int64_t)g.T + g.d - 1) / g.d;
    g.lc = L > 0 ? (int32_t)((L + nch - 1) / nch) : 1;  // an empty sequence has no chunks
    g.nch = (int32_t)((L + g.lc - 1) / g.lc);
    g.items = (size_t)g.nch * g.d * g.M;
}

// The shared walk plan: a grid of about three waves per SIMD (256 CUs x 4
// SIMDs), chunks of each residue class such that each thread has two or three
// items (each chunk at least 2k steps)
constexpr int64_t kBnTarget = 256 * 4 * 3 * 64;
inline void bn_plan(BnGeom& g)
{
    const int64_t L = ((int64_t)g.T + g.d - 1) / g.d;
    const int64_t walks = (int64_t)g.M * g.d;
    int64_t nch = walks > 0 ? (2 * kBnTarget + walks - 1) / walks : 1;
    const int64_t max_nch = L / (2 * (int64_t)g.k);
    nch = nch < max_nch ? nch : max_nch;
    bn_chunks(g, nch > 1 ? nch : 1);
    bn_threads(g, kBnTarget);
}

// Estimated time of the backward walk, in steps of one wave's issue: two waves
// per SIMD are resident, a SIMD's last wave alone takes as long as two, and a
// cut class repeats k-1 steps per cut (three quarters of their work).
inline double bn_backward_cost(const BnGeom& g)
{
    const int64_t W = (int64_t)g.G / 64, slots = 2 * 1024;
    const int64_t rounds = (W + slots - 1) / slots, per = ((int64_t)g.items + g.G - 1) / (int64_t)g.G;
    return 2.0 * rounds * per * (g.lc + 0.75 * (g.k - 1) * (g.nch - 1) / g.nch + 8.0);
}

// The backward's plan.  At orders 15 to 22 its walk holds 176 to 248 VGPRs, so
// two waves per SIMD are resident and the shared plan's three leave a second
// round that is mostly empty.  There the fewest threads of shortest estimated
// time are taken among the numbers of chunks, never more threads than the
// shared plan has: the workspace is sized by it.  It is taken where the estimate
// falls to 0.77 of the shared plan's: of 162 layers (11 shapes, orders 15 to 22,
// d = 1 to 3) the 78 with 0.42 to 0.75 took 0.72 to 1.00 of its time, 0.91 on
// average, and those at 0.79 and 0.80 ([128,64,100,13] d = 2) 1.05 and 1.00.
// Lower orders hold three waves or more; above 22 the walk spills and one is
// resident, unmeasured.
inline void bn_backward_plan(BnGeom& g)
{
    if (g.k < 15 || g.k > 22 || g.items == 0)
        return;
    BnGeom best = g;
    double least = 0.77 * bn_backward_cost(g);
    const int64_t L = ((int64_t)g.T + g.d - 1) / g.d;
    for (int64_t nch = 1; nch == 1 || (nch <= 64 && nch * 2 * g.k <= L); ++nch)
        for (int rounds = 1; rounds <= 2; ++rounds) {
            BnGeom t = g;
            bn_chunks(t, nch);
            bn_threads(t, (int64_t)rounds * 2 * 1024 * 64);
            const double cost = bn_backward_cost(t);
            if (t.G <= g.G && cost < least) {
                least = cost;
                best = t;
            }
        }
    g = best;
}

size_t bn_workspace_bytes(const BnGeom& g);
hipError_t launch_bn_forward_stats(const BnGeom& g, const float* x, const float* w, const float* gamma,
                                   const float* beta, float eps, float* w_f, float* b_f, double* aux,
                                   double* stats, void* workspace, hipStream_t stream);
hipError_t launch_bn_backward(const BnGeom& g, const float* x, const float* w, const double* aux, float eps,
                              const float* grad_wf, const float* grad_bf, float* grad_x, float* grad_w,
                              float* grad_gamma, float* grad_beta, void* workspace, hipStream_t stream);

}  // namespace mfpsn
