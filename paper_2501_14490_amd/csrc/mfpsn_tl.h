// Internal interface of the time-last kernels for the C-ABI layer: the tiles of
// mfpsn_tl_tile.hip, and the forward for the longest histories (mfpsn_tl.hip).
// Not installed; not part of the ABI.
#pragma once

#include <hip/hip_runtime_api.h>
#include <stdint.h>

#include "mfpsn_tl_tile.h"

namespace mfpsn {

constexpr int kTlWaves = 4;                 // waves per block
constexpr int kTlMaxHalo = 2048;            // longest history tl_fwd_kernel stages in LDS
// What sizes the backward's workspace (tl_bwd_slots)
constexpr int kTlShortT = 64;               // longest column counted per 64 columns
constexpr int kTlSeg = 256;                 // steps per counted segment of longer columns
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
    int32_t steps_per_lane; // tl_fwd_kernel: 1 or 4: segments of 64 or 256 time steps
    int32_t nseg;           // tl_fwd_kernel: segments per column, ceil(T / (64 * steps_per_lane))
    int32_t halo;           // tl_fwd_kernel: LDS history slots per wave (0: taps read from global memory)
    int32_t shift_lo, shift_hi;
    float v_th;
    int32_t v_th_q;
    float fast_lo, fast_hi; // range of |x| in which the exponent-add tap is exact
    int32_t vec_x;          // x is 16-byte aligned
    int32_t vec_s;          // spikes are 16-byte aligned
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
                            // channel, at tile_slot
    int64_t M;              // columns, N*C*S
    int32_t T, C, S, k, d;
    int32_t shift_lo, shift_hi;
    float v_th;
    int32_t v_th_q;
    int32_t sg;             // surrogate kind
    float alpha;
    float fast_lo, fast_hi; // range of |x| and |dH| in which the exponent-add tap is exact
    int32_t vec_x;          // x, g and grad_x are 16-byte aligned
    int64_t chunk;          // tiles per wave (set by the launcher)
    int32_t x_exact;        // as TlArgs::x_exact
};

// Slots of partial sums the backward's workspace holds (k + 1 sums each):
// for columns up to kTlShortT steps one per 64 columns and one per (n, c) row,
// else one per channel and four per four segments of kTlSeg (kTlSegLong)
// steps, at most kTlMaxWaves.  The tile plan keeps within them.
inline int64_t tl_bwd_slots(int64_t M, int32_t T, int32_t C, int32_t N, int64_t span)
{
    if (M == 0 || T == 0)
        return 0;
    if (T <= kTlShortT)
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

// One storage type's launchers, each in its own translation unit
void tl_forward_f32(const TlArgs& a, hipStream_t st);
void tl_forward_bf16(const TlArgs& a, hipStream_t st);
void tl_forward_q88(const TlArgs& a, hipStream_t st);

}  // namespace mfpsn
