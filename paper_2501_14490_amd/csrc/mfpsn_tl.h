// Internal interface of the time-last kernels for the C-ABI layer: the tiles of
// mfpsn_tl_tile.hip, and the kernels of mfpsn_tl.hip: a lane per column for
// short columns, and the forward for the longest histories.
// Not installed; not part of the ABI.
#pragma once

#include <hip/hip_runtime_api.h>
#include <stdint.h>

#include "mfpsn_tl_tile.h"

namespace mfpsn {

constexpr int kTlWaves = 4;                 // waves per block
constexpr int kTlMaxHalo = 2048;            // longest history tl_fwd_kernel stages in LDS
constexpr int kTlSteps = 4;                 // steps per lane of its segments
constexpr int kTlColsMaxT = 64;             // longest column of the lane-per-column kernels
// What sizes the backward's workspace (tl_bwd_slots)
constexpr int kTlSeg = 256;                 // steps per counted segment of columns above kTlColsMaxT
constexpr int kTlSegLong = 1024;            // the same for histories (k-1) d above 64
constexpr int kTlMaxWaves = 32768;          // most waves counted

struct TlArgs {
    const void* x;          // [N][C][S][T] storage type
    const int8_t* sign;     // [C][k]
    const int8_t* shift;    // [C][k]
    const void* bias;       // float[C] or int32[C]
    uint8_t* spikes;        // [N][C][S][T]
    void* h_out;            // nullable, float or int32 [N][C][S][T]
    int64_t M;              // columns, N*C*S
    int32_t T, C, S, k, d;
    int32_t nseg;           // tl_fwd_kernel: segments of 64 kTlSteps steps per column
    int32_t halo;           // tl_fwd_kernel: LDS history slots per wave (0: taps read from global memory)
    int32_t shift_lo, shift_hi;
    float v_th;
    int32_t v_th_q;
    float fast_lo, fast_hi; // range of |x| in which the exponent-add tap is exact
    uint32_t tdiv;          // columns: floor(2^32 / T) + 1 (T >= 2; 0 when T = 1): e / T = umulhi(e, tdiv) for e < 64 T
    int32_t vec_x;          // x is 4-byte aligned (columns: to 4 elements)
    int32_t vec_s;          // spikes are 16-byte aligned
    int32_t vec_h;          // h_out is 16-byte, spikes are 4-byte aligned
    int32_t x_exact;        // every stored input has exact tap products (as Geom::x_exact)
};

hipError_t launch_forward_time_last(const TlArgs& a, int dtype, hipStream_t stream);

// Backward in the time-last layout
struct TlBwdArgs {
    const void* x;          // [N][C][S][T] storage type
    const void* g;          // grad_spikes, [N][C][S][T] storage type
    const int8_t* sign;     // [C][k]
    const int8_t* shift;    // [C][k]
    const void* bias;       // float[C] or int32[C]
    void* grad_x;           // [N][C][S][T] float, bfloat16 bits or int32
    void* part;             // [slots][k+1] double (float data) or int64 (Q8.8): sums of one wave and
                            // channel, at tile_slot (columns: of one block and (n, c) row, at block + row)
    int64_t M;              // columns, N*C*S
    int32_t T, C, S, k, d;
    int32_t shift_lo, shift_hi;
    float v_th;
    int32_t v_th_q;
    int32_t sg;             // surrogate kind
    float alpha;
    float fast_lo, fast_hi; // range of |x| and |dH| in which the exponent-add tap is exact
    uint32_t tdiv;          // as TlArgs::tdiv
    int32_t vec_x;          // x and g are 4-byte aligned (columns: to 4 elements)
    int32_t vec_o;          // tiles: grad_x is 16-byte aligned (bf16: 8-byte)
    int64_t chunk;          // tiles per wave (set by the launcher)
    int32_t x_exact;        // as TlArgs::x_exact
};

// Slots of partial sums the backward's workspace holds (k + 1 sums each):
// for columns up to kTlColsMaxT steps one per 64 columns and one per (n, c) row,
// else one per channel and four per four segments of kTlSeg (kTlSegLong)
// steps, at most kTlMaxWaves.  The tile plan keeps within them.
inline int64_t tl_bwd_slots(int64_t M, int32_t T, int32_t C, int32_t N, int64_t span)
{
    if (M == 0 || T == 0)
        return 0;
    if (T <= kTlColsMaxT)
        return (M + 63) / 64 + (int64_t)N * C;
    const int seg = span > 64 ? kTlSegLong : kTlSeg;
    const int64_t waves = (M * ((T + seg - 1) / seg) + kTlWaves - 1) / kTlWaves * kTlWaves;
    return (waves < kTlMaxWaves ? waves : kTlMaxWaves) + C;
}

// The tile kernels (mfpsn_tl_tile.hip).  The backward writes its partial sums
// to the `slots` slots of a.part and adds each channel's in a fixed order into
// grad_w and grad_b.
hipError_t launch_forward_tiles(const TlArgs& a, const TileGeom& g, int dtype, hipStream_t stream);
hipError_t launch_backward_tiles(TlBwdArgs& a, const TileGeom& g, int64_t slots, int dtype, void* grad_w, void* grad_b,
                                 hipStream_t stream);
// One storage type's launchers for the orders from KLO up to the next entry
constexpr int kTileKs[4] = {1, 9, 17, 25};
template <int DT, int KLO> hipError_t tile_forward(const TlArgs& a, const TileGeom& g, hipStream_t stream);
template <int DT, int KLO>
hipError_t tile_backward(TlBwdArgs& a, const TileGeom& g, int64_t slots, hipStream_t stream);

// Whether a call on columns of T <= kTlColsMaxT steps goes to the
// lane-per-column kernels.  A tile has at most 64 / d columns and starts anew
// for each, a column's block takes 64 columns whatever d; against that a tile
// spreads a column over lanes, so it wins where columns are long, dilations
// small or lanes scarce, and the column backward loses most of its waves to
// registers at high orders.  Fitted on MI355X to 9615 calls of both kernels (T
// 1 to 64, all orders, d 1 to 32, 2^16 to 2^24 elements): the forwards that go
// to tiles (2583) take 0.76 of the columns' time on average, the backwards (4244)
// 0.67, and the worst of them 1.15 and 1.17.  Columns / tiles, us, 2^24 elements,
// k = 8: bf16 T = 30, d = 1, 3 forward 19, 20 / 20, 27, backward 69, 68 / 63, 77;
// bf16 T = 64, d = 1 30 / 21 and 93 / 69; f32 T = 32, d = 1 24 / 24 and 90 / 68.
// 512 columns of 64 steps, f32 k = 16 backward 39 / 17.
struct TlColumnsRule {
    int32_t few_t;      // few columns (at most few_cols): tiles from this length
    int64_t few_cols;
    int32_t t0, per_d;  // more: from (t0 + per_d d) / 2 steps
    int32_t steps;      // and with as many steps per residue class
    int32_t max_k;      // up to this order
    // and these numbers of columns, orders and lengths, with as many as `steps`
    // per class (max_k 0: none)
    struct {
        int32_t min_cols, max_cols, min_k, max_k, min_t, max_t, steps;
    } also[8];
};
constexpr int32_t kTlMany = INT32_MAX;  // no upper limit of columns
constexpr TlColumnsRule kTlColumnsRule[2][3] = {
    // forward: f32, bf16, Q8.8
    {{30, 32768, 84, 4, 4, 32, {{1 << 17, kTlMany, 2, 16, 40, 64, 12}, {1 << 17, kTlMany, 22, 32, 40, 64, 7}}},
     {32, 49152, 108, 5, 4, 25, {{0, 32768, 2, 32, 28, 64, 2}, {1 << 20, kTlMany, 30, 32, 1, 64, 6}}},
     {28, 32768, 80, 12, 3, 22, {{0, 32768, 18, 32, 20, 64, 2}, {1 << 18, kTlMany, 32, 32, 1, 64, 4},
         {1 << 17, kTlMany, 2, 12, 40, 64, 14}}}},
    // backward
    {{36, 6553, 48, 6, 5, 14, {{0, 4096, 2, 32, 8, 64, 12}, {0, 32768, 2, 24, 56, 64, 12},
         {1 << 17, kTlMany, 26, 32, 1, 64, 8}, {1 << 17, kTlMany, 9, 32, 40, 64, 8},
         {1 << 19, kTlMany, 26, 32, 4, 32, 3}, {1 << 15, kTlMany, 2, 11, 28, 64, 5},
         {1 << 18, kTlMany, 18, 32, 4, 24, 6}, {1 << 15, kTlMany, 2, 16, 40, 64, 6}}},
     {48, 6553, 96, 4, 4, 16, {{0, 32768, 2, 12, 8, 64, 12}, {0, 4096, 2, 32, 8, 64, 12},
         {1 << 17, kTlMany, 26, 32, 1, 64, 6}, {1 << 19, kTlMany, 26, 32, 4, 24, 2},
         {1 << 18, kTlMany, 16, 24, 4, 24, 6}, {1 << 15, kTlMany, 12, 16, 20, 40, 14},
         {1 << 15, kTlMany, 26, 32, 40, 64, 2}}},
     {48, 16384, 36, 6, 4, 17, {{0, 32768, 2, 12, 8, 64, 12}, {0, 4096, 2, 32, 20, 64, 2},
         {1 << 18, kTlMany, 22, 32, 1, 64, 4}, {1 << 17, kTlMany, 9, 32, 1, 64, 12},
         {1 << 15, kTlMany, 18, 32, 40, 64, 2}, {1 << 19, kTlMany, 22, 32, 4, 16, 2},
         {1 << 17, kTlMany, 22, 32, 20, 64, 2}, {1 << 20, kTlMany, 12, 20, 4, 16, 3}}}},
};

inline bool tl_by_columns(bool backward, int dtype, int64_t M, int32_t T, int32_t k, int32_t d)
{
    if (T > kTlColsMaxT)
        return false;
    const TlColumnsRule& r = kTlColumnsRule[backward ? 1 : 0][dtype];
    for (const auto& c : r.also)
        if (M >= c.min_cols && M <= (c.max_cols == kTlMany ? M : c.max_cols) && k >= c.min_k && k <= c.max_k &&
            T >= c.min_t && T <= c.max_t && T >= (int64_t)c.steps * d)
            return false;
    if (k > r.max_k || T < (int64_t)r.steps * d)
        return true;
    return M <= r.few_cols ? T < r.few_t : 2 * T < r.t0 + (int64_t)r.per_d * d;
}

// Whether a short tile backward is worth it although its slots of partial sums
// keep it from waves that fit (tile_short_of_waves): f32 and Q8.8 columns of 42
// steps and more at orders up to 12 take 0.71 of the columns' time (of 450 calls
// the worst 1.1), others 1.0 to 1.7.
inline bool tl_bears_few_waves(int dtype, int32_t T, int32_t k, int32_t d)
{
    return T > kTlColsMaxT || (dtype != 1 && T >= 42 && T >= (int64_t)4 * d && k <= 12);
}

// The lane-per-column kernels (mfpsn_tl.hip, T <= kTlColsMaxT).  The backward
// as launch_backward_tiles, with a slot for each block and (n, c) row that share
// a column.
hipError_t launch_forward_cols(const TlArgs& a, int dtype, hipStream_t stream);
hipError_t launch_backward_cols(const TlBwdArgs& a, int dtype, void* grad_w, void* grad_b, hipStream_t stream);

// The same of one storage type for the orders from KLO up to the next of kTileKs
template <int DT, int KLO> void tl_forward(const TlArgs& a, hipStream_t st);
template <int DT, int KLO> void tl_cols_forward(const TlArgs& a, hipStream_t st);
template <int DT, int KLO> void tl_cols_backward(const TlBwdArgs& a, hipStream_t st);

}  // namespace mfpsn
