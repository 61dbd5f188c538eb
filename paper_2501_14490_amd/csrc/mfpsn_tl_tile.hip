// gfx950 kernels of the mul-free channel-wise neuron (arXiv 2501.14490,
// Eqs. mfdpsn_charge, mfdpsn_fire; App. A.3 Eqs. backward_X, backward_W,
// backward_b) for the time-last layout [N][C][S][T]: a wave per tile of whole
// columns, or of one long segment of a column (mfpsn_tl_tile.h).
//
// A tile's inputs are contiguous in memory.  They are copied to LDS as they
// lie, 16 bytes per lane and access, and the 64 lanes walk them there: a lane
// takes one residue class of the dilation of one column, or a chunk of it,
// with the last k values in a register ring (a compile-time slot per step
// inside blocks of k unrolled steps), so a step reads one input from LDS
// however high the order is.  What these kernels wait for is VALU issue (the
// taps and the surrogate), as in the time-first layout, not the transposition:
// the layout costs two LDS accesses per value.
//
// Forward: spikes go to a byte image in LDS that is stored with 16-byte
// accesses.  Backward, two walks: the first, in ascending time, recomputes H
// and turns each grad_spikes value in LDS into dH = g sigma'(H - V_th), adding
// the exact products x dH to the lane's grad_w sums; the second, in
// descending time, gathers grad_x[t] = sum_i w_i dH[t + (k-1-i) d] from a
// ring of dH and writes it over dH[t], which no other lane needs any more
// (the values a chunk needs from the next one are read before any is
// written).  Both sums run in ascending tap order, as in the definition.
// Waves take contiguous runs of tiles that share channels, so taps and
// grad_w sums stay in registers, and the sums are reduced once per run.
//
// Measured on MI355X (forward + backward, us), against a lane per column of a
// transposed tile up to T = 64 and a lane per time step of a segment above, which
// read k values from LDS per step: f32 [32,128,256,32] k = 8 208 -> 152 (its
// forward, 25, by columns), f32 [250,256,512] k = 16 d = 2 570 -> 235, Q8.8
// [4096,16,1024] k = 32 d = 4 1655 -> 733.  The backward issues 88 to 150 VALU
// instructions per 64 elements at orders 8 and 16 and keeps the VALUs about 85%
// busy; LDS bank conflicts are below 2% of the time.
// Short columns go to tiles only where they are faster (tl_by_columns): a lane
// takes one class, so a tile has at most 64 / d columns, whose start costs as
// much as the few steps of a short one.
//
// The arithmetic is that of mfpsn_kernels.hip: a float tap is a fused
// multiply-add by sign 2^-shift where every value of the tile has exact
// products, else a product and an add (always right: the product rounds as
// the exponent move does); a Q8.8 tap is a floor shift and an xor-add.
// Values before time 0 and past the end are zeros, whose terms change no bit.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <atomic>
#include <type_traits>
#include <utility>

#include "mfpsn.h"
#include "mfpsn_surrogate.h"
#include "mfpsn_tl.h"

namespace mfpsn {
namespace {

typedef uint32_t V4 __attribute__((ext_vector_type(4)));

// Storage types: V the value in registers, E the element in memory and in
// the image of x, kV elements per 16 bytes
template <int DT> struct TileIO;
template <> struct TileIO<MFPSN_F32> {
    using V = float;
    using E = float;
    using W = double;
    static __device__ __forceinline__ V get(E e) { return e; }
};
template <> struct TileIO<MFPSN_BF16> {
    using V = float;
    using E = uint16_t;
    using W = double;
    static __device__ __forceinline__ V get(E e) { return __builtin_bit_cast(float, (uint32_t)e << 16); }
};
template <> struct TileIO<MFPSN_Q8_8> {
    using V = int32_t;
    using E = int16_t;
    using W = int64_t;
    static __device__ __forceinline__ V get(E e) { return e; }
};

// LDS writes of every lane of the wave before any lane reads (a wave's LDS
// operations run in order; this keeps the compiler from moving them)
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// 16-byte pieces of a tensor from element e0 (a multiple of 16 bytes) to its
// end; the 4-byte words of a piece that are not wholly inside read as zeros
__device__ __forceinline__ __amdgpu_buffer_rsrc_t pieces(const void* p, int64_t e0, int64_t total, int es)
{
    const uint64_t rem = (uint64_t)(total - e0) * es;
    const int n = (int)(rem > 0x7FFFFFF0ull ? 0x7FFFFFF0ull : rem);
    return __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)p + (uint64_t)e0 * es), (short)0, n, 0x00020000);
}

// The smallest magnitude among the checked values, zero apart: 2 |v| - 1 in
// the bit patterns, which zero wraps to the largest
__device__ __forceinline__ uint32_t mag_key(float v) { return 2u * __builtin_bit_cast(uint32_t, v) - 1u; }

// Whether the tap products of the values seen are all exact.  Only their
// lower bound is followed: with negative shifts (products that can grow) the
// callers take the rounded products without looking.
struct ExactCheck {
    uint32_t least = 0xFFFFFFFFu;
    __device__ __forceinline__ void see(float v)
    {
        const uint32_t m = mag_key(v);
        least = least < m ? least : m;
    }
    __device__ __forceinline__ bool inexact(float lo) const { return least < mag_key(lo); }
};

// Makes v opaque here, so that integer sums are not reassociated (a tap is then
// one shift and one xor-add, a grad_w term one multiply-add)
template <typename T> __device__ __forceinline__ void pin(T& v) { asm volatile("" : "+v"(v)); }

// The k taps of the lane's channel
template <int DT, int K> struct TileTaps {
    static constexpr bool kF = DT != MFPSN_Q8_8;
    using V = typename TileIO<DT>::V;
    float w[kF ? K : 1];
    int sh[kF ? 1 : K], neg[kF ? 1 : K];
    int nneg;
    __device__ __forceinline__ void load(const int8_t* sign, const int8_t* shift, int c, int lo, int hi)
    {
        nneg = 0;
#pragma unroll
        for (int i = 0; i < K; ++i) {
            int s = shift[(int64_t)c * K + i];
            s = s < lo ? lo : (s > hi ? hi : s);
            const bool n = sign[(int64_t)c * K + i] < 0;
            if constexpr (kF) {
                w[i] = __builtin_bit_cast(float, ((uint32_t)(127 - s) << 23) | (n ? 0x80000000u : 0u));
            } else {
                sh[i] = s;
                neg[i] = n ? -1 : 0;
                nneg += n ? 1 : 0;
            }
        }
    }
    // what a sum over all k taps starts from (Q8.8: the -1 of every negative
    // tap's xor)
    __device__ __forceinline__ V start() const { return kF ? V(0) : V(nneg); }
    template <bool EXACT> __device__ __forceinline__ V add(V acc, V in, int i) const
    {
        if constexpr (!kF) {
            V sum = ((in >> sh[i]) ^ neg[i]) + acc;
            pin(sum);
            return sum;
        } else if constexpr (EXACT) {
            return acc + in * w[i];
        } else {
            return __builtin_fmaf(in, w[i], acc);
        }
    }
};

// Element of a row's first step in an image whose rows are `stride` elements
// apart: a piece's element e (counted from the tile's first) lies in row e / T
__device__ __forceinline__ int row_shift(const TileGeom& g, int e, int stride)
{
    return stride != g.T ? (int)__umulhi((uint32_t)e, g.tdiv) * (stride - g.T) : 0;
}

// Four words to or from an image, whole 16-byte pieces unless rows are padded
__device__ __forceinline__ void put4(char* p, V4 w, bool padded)
{
    if (!padded) {
        *(V4*)p = w;
    } else {
#pragma unroll
        for (int j = 0; j < 4; ++j)
            ((uint32_t*)p)[j] = w[j];
    }
}
__device__ __forceinline__ V4 get4(const char* p, bool padded)
{
    if (!padded)
        return *(const V4*)p;
    V4 w;
#pragma unroll
    for (int j = 0; j < 4; ++j)
        w[j] = ((const uint32_t*)p)[j];
    return w;
}

// Copies `count` elements from element e0 of src into the LDS image img (from
// its element e0 mod kV, so that 16-byte pieces stay 16-byte pieces) and,
// with PAIR, `count2` from f0 of src2 into img2, widened to 32 bits; the loads
// of up to U pieces of each are issued before the first LDS write.  off and
// off2 get the offsets of the first elements.  The 16-byte buffer loads need
// 4-byte alignment; 16-bit tensors off it (vec = 0) go element by element.  With CHECK, the values of src go to chk.
template <int DT, bool PAIR, bool CHECK, int U>
__device__ __forceinline__ void stage(const TileGeom& g, const void* src, int64_t e0, int count, const void* src2,
                                      int64_t f0, int count2, int64_t total, bool vec, char* img, char* img2,
                                      ExactCheck& chk, int& off, int& off2)
{
    using E = typename TileIO<DT>::E;
    using V = typename TileIO<DT>::V;
    constexpr int es = (int)sizeof(E), kV = 16 / es;
    const int lane = (int)threadIdx.x;
    const bool xpad = g.xs != g.T, opad = PAIR && g.os != g.T;
    if (!vec) {
        off = off2 = 0;
        for (int i = lane; i < count; i += 64) {
            const E e = ((const E*)src)[e0 + i];
            ((E*)img)[i + row_shift(g, i, g.xs)] = e;
            if constexpr (CHECK)
                chk.see(TileIO<DT>::get(e));
        }
        if constexpr (PAIR)
            for (int i = lane; i < count2; i += 64)
                ((V*)img2)[i + row_shift(g, i, g.os)] = TileIO<DT>::get(((const E*)src2)[f0 + i]);
        return;
    }
    // (padded rows are whole pieces, or for the widened image whole half
    // pieces: off is 0, off2 is 0 or 4)
    off = (int)(e0 & (kV - 1));
    off2 = PAIR ? (int)(f0 & (kV - 1)) : 0;
    const auto rs = pieces(src, e0 - off, total, es);
    const auto rs2 = PAIR ? pieces(src2, f0 - off2, total, es) : rs;
    const int n = (off + count + kV - 1) / kV, n2 = PAIR ? (off2 + count2 + kV - 1) / kV : 0;
    const int top = n > n2 ? n : n2;
    // four 32-bit values of src2's elements e .. e + 3 (from the tile's first)
    auto put_wide = [&](int e, V4 w) __attribute__((always_inline)) {
        if (!opad)
            *(V4*)(img2 + 4 * (off2 + e)) = w;
        else if (e >= 0 && e < count2)
            put4(img2 + 4 * (off2 + e + row_shift(g, e, g.os)), w, true);
    };
    for (int b = 0; b < top; b += 64 * U) {
        V4 r[U], s[U];
#pragma unroll
        for (int u = 0; u < U; ++u)
            r[u] = __builtin_amdgcn_raw_buffer_load_b128(rs, 16 * (b + lane + 64 * u), 0, 0);
        if constexpr (PAIR) {
#pragma unroll
            for (int u = 0; u < U; ++u)
                s[u] = __builtin_amdgcn_raw_buffer_load_b128(rs2, 16 * (b + lane + 64 * u), 0, 0);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int q = b + lane + 64 * u;
            if (q < n) {
                put4(img + 16 * q + es * row_shift(g, kV * q, g.xs), r[u], xpad);
                if constexpr (CHECK) {
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        if constexpr (DT == MFPSN_F32) {
                            chk.see(__builtin_bit_cast(float, (uint32_t)r[u][j]));
                        } else if constexpr (DT == MFPSN_BF16) {
                            chk.see(__builtin_bit_cast(float, (uint32_t)r[u][j] << 16));
                            chk.see(__builtin_bit_cast(float, (uint32_t)r[u][j] & 0xFFFF0000u));
                        }
                    }
                }
            }
            if constexpr (PAIR) {
                if (q < n2) {
                    if constexpr (DT == MFPSN_F32) {
                        put_wide(kV * q - off2, s[u]);
                    } else {
                        V4 a, c;
#pragma unroll
                        for (int j = 0; j < 4; ++j) {
                            const uint32_t w = s[u][j];
                            const uint32_t lo = DT == MFPSN_BF16 ? w << 16 : (uint32_t)((int32_t)(w << 16) >> 16);
                            const uint32_t hi = DT == MFPSN_BF16 ? w & 0xFFFF0000u : (uint32_t)((int32_t)w >> 16);
                            if (j < 2) {
                                a[2 * j] = lo;
                                a[2 * j + 1] = hi;
                            } else {
                                c[2 * j - 4] = lo;
                                c[2 * j - 3] = hi;
                            }
                        }
                        put_wide(kV * q - off2, a);
                        put_wide(kV * q - off2 + 4, c);
                    }
                }
            }
        }
    }
    if constexpr (es == 2) {
        // the last element of an odd tensor lies in a word that reads as zeros
        // (padded rows are even, and so is their tensor)
        if ((total & 1) != 0 && lane == 0) {
            if (e0 + count == total) {
                const E e = ((const E*)src)[total - 1];
                ((E*)img)[off + count - 1] = e;
                if constexpr (CHECK)
                    chk.see(TileIO<DT>::get(e));
            }
            if (PAIR && f0 + count2 == total)
                ((V*)img2)[off2 + count2 - 1] = TileIO<DT>::get(((const E*)src2)[total - 1]);
        }
    }
}

// Stores elements [0, count) of a tile's image (element 0 at off, rows of T
// elements `stride` apart) to dst from its element d0 (d0 - off is a multiple
// of a piece when vec): whole 16-byte pieces of the image at once and the ends
// element by element, each value through out() (bf16: rounded).
template <typename I, typename E>
__device__ __forceinline__ void unstage(const TileGeom& g, const I* img, int off, int count, int stride, E* dst,
                                        int64_t d0, bool vec)
{
    // elements per group: a piece of the image, or of dst where dst is narrower
    constexpr bool kNarrow = sizeof(E) < sizeof(I);
    constexpr int kV = 16 / (int)sizeof(I);
    const int lane = (int)threadIdx.x;
    const bool padded = stride != g.T;
    auto value = [&](int e) __attribute__((always_inline)) {
        const I v = img[off + e + row_shift(g, e, stride)];
        if constexpr (kNarrow)
            return __builtin_bit_cast(E, (__bf16)v);
        else
            return v;
    };
    if (!vec) {
        for (int i = lane; i < count; i += 64)
            dst[d0 + i] = value(i);
        return;
    }
    const int q0 = (off + kV - 1) / kV, q1 = (off + count) / kV;  // whole pieces of the image
    E* base = dst + (d0 - off);
    for (int q = q0 + lane; q < q1; q += 64) {
        const V4 w = get4((const char*)(img + kV * q + (padded ? row_shift(g, kV * q - off, stride) : 0)), padded);
        if constexpr (kNarrow) {
            typedef uint32_t V2 __attribute__((ext_vector_type(2)));
            V2 h;
#pragma unroll
            for (int j = 0; j < 2; ++j)
                h[j] = (uint32_t)__builtin_bit_cast(uint16_t, (__bf16)__builtin_bit_cast(float, (uint32_t)w[2 * j])) |
                       (uint32_t)__builtin_bit_cast(uint16_t, (__bf16)__builtin_bit_cast(float, (uint32_t)w[2 * j + 1]))
                           << 16;
            __builtin_nontemporal_store(h, (V2*)base + q);
        } else {
            __builtin_nontemporal_store(w, (V4*)base + q);
        }
    }
    const int head = min(q0 * kV - off, count);
    if (lane < head)
        base[off + lane] = value(lane);
    const int t0 = q1 * kV - off, tail = count - t0;  // (no whole piece, and t0 below 0: the head has it all)
    if (q1 >= q0 && lane < tail)
        base[off + t0 + lane] = value(t0 + lane);
}

// As unstage, for an image of potentials: stores them to h and the spikes they
// are to spikes, four at once (rows of padded images are whole groups of four).
template <typename V>
__device__ __forceinline__ void unstage_h(const TileGeom& g, const V* img, int off, int count, V v_th, V* h,
                                          uint8_t* spikes, int64_t d0, bool vec)
{
    const int lane = (int)threadIdx.x;
    const bool padded = g.os != g.T;
    auto one = [&](int e) __attribute__((always_inline)) {
        const V v = img[off + e + row_shift(g, e, g.os)];
        h[d0 + e] = v;
        spikes[d0 + e] = v >= v_th ? 1 : 0;
    };
    if (!vec) {
        for (int i = lane; i < count; i += 64)
            one(i);
        return;
    }
    const int q0 = (off + 3) / 4, q1 = (off + count) / 4;  // whole groups
    for (int q = q0 + lane; q < q1; q += 64) {
        const V4 w = get4((const char*)(img + 4 * q + (padded ? row_shift(g, 4 * q - off, g.os) : 0)), padded);
        uint32_t s = 0;
#pragma unroll
        for (int j = 0; j < 4; ++j)
            s |= (__builtin_bit_cast(V, (uint32_t)w[j]) >= v_th ? 1u : 0u) << (8 * j);
        __builtin_nontemporal_store(w, (V4*)(h + (d0 - off)) + q);
        __builtin_nontemporal_store(s, (uint32_t*)(spikes + (d0 - off)) + q);
    }
    const int head = min(q0 * 4 - off, count);
    if (lane < head)
        one(lane);
    const int t0 = q1 * 4 - off, tail = count - t0;  // (no whole group, and t0 below 0: the head has it all)
    if (q1 >= q0 && lane < tail)
        one(t0 + lane);
}

// a / b, with a 32-bit division where both fit one (most of a tile's start on few
// columns was 64-bit divisions)
__device__ __forceinline__ int64_t divide(int64_t a, int64_t b)
{
    return ((uint64_t)(a | b) >> 32) == 0 ? (int64_t)((uint32_t)a / (uint32_t)b) : a / b;
}

// The tiles of a wave in turn: columns col0 .. col0 + rows - 1 of group p,
// steps from t0 (all wave-uniform; the divisions are done once)
struct Cursor {
    int64_t col0;
    int p, n, blk, seg, rows, t0;
    __device__ __forceinline__ void set(const TileGeom& g)
    {
        t0 = seg * g.seg;
        if (g.by_channel) {
            col0 = ((int64_t)n * g.C + p) * g.S + (int64_t)blk * g.G;
            rows = min(g.G, g.S - blk * g.G);
        } else {
            const int64_t SC = (int64_t)g.S * g.C, j0 = (int64_t)p * g.G;
            col0 = n * SC + j0;
            rows = (int)min((int64_t)g.G, SC - j0);
        }
    }
    __device__ __forceinline__ Cursor(const TileGeom& g, int64_t q)
    {
        p = (int)divide(q, g.Z);
        const uint32_t z = (uint32_t)(q - (int64_t)p * g.Z), per = (uint32_t)(g.sblk * g.nseg);
        n = (int)(z / per);
        const uint32_t rest = z - (uint32_t)n * per;
        blk = (int)(rest / (uint32_t)g.nseg);
        seg = (int)(rest - (uint32_t)blk * (uint32_t)g.nseg);
        set(g);
    }
    __device__ __forceinline__ void next(const TileGeom& g, int N)
    {
        if (++seg == g.nseg) {
            seg = 0;
            if (++blk == g.sblk) {
                blk = 0;
                if (++n == N) {
                    n = 0;
                    ++p;
                }
            }
        }
        set(g);
    }
    // this tile's place in its group
    __device__ __forceinline__ int64_t z(const TileGeom& g) const
    {
        return ((int64_t)n * g.sblk + blk) * g.nseg + seg;
    }
};

// The lane's part of a window of W steps: class steps [j0, j1) of class r
// (times r + j d, from the window's start), L steps in the class; R = tile_chunk(g, W)
struct Part {
    int r, j0, j1, L;
};
__device__ __forceinline__ Part part_of(const TileGeom& g, int W, int r, int chunk, int R)
{
    Part a;
    a.r = r;
    a.L = r < W ? (int)((uint32_t)(W - r + g.d - 1) / (uint32_t)g.d) : 0;
    a.j0 = min(chunk * R, a.L);
    a.j1 = min(a.j0 + R, a.L);
    return a;
}

// steps 0 .. top - 1 of a walk in blocks of K, step u of a block on the
// lanes with steps left (n of the lane)
template <int K, typename Step> __device__ __forceinline__ void walk_steps(int top, int n, Step&& step)
{
    for (int b = 0; b < top; b += K) {
        [&]<int... U>(std::integer_sequence<int, U...>) __attribute__((always_inline)) {
            (void)((b + U < top ? ((b + U < n ? step(std::integral_constant<int, U>{}) : void()), true) : false) &&
                   ...);
        }(std::make_integer_sequence<int, K>{});
    }
}

// WANT_H: the second image holds H (4 bytes per element), from which H and the
// spikes are stored as they lie in memory, else the spikes.  Stored by the lanes
// as they walk, 64 scattered values per step, H took 131 us for f32
// [512,16,64,32] k = 4 d = 1 and 85 us for T = 1000 k = 8 d = 1 (2^24 elements);
// from the image 47 and 44 (two passes over the image beside the 4 bytes more).
template <int DT, int K, bool WANT_H>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(K <= 16 ? 4 : 3))) void tile_fwd_kernel(
    TlArgs a, TileGeom g, int64_t chunk)
{
    using IO = TileIO<DT>;
    using V = typename IO::V;
    using E = typename IO::E;
    constexpr bool kF = DT != MFPSN_Q8_8;
    constexpr int es = (int)sizeof(E), os = WANT_H ? 4 : 1;
    extern __shared__ __attribute__((aligned(16))) char lds[];
    char* xi = lds;
    char* oi = lds + g.lds_x;
    const int xstep = g.d * es;
    const int lane = (int)threadIdx.x;
    const int row = min(lane / g.Q, g.G - 1), q = lane - row * g.Q;
    const bool mine = q < g.ncls * g.m && lane < g.G * g.Q;
    const int64_t total = a.M * a.T;
    int64_t t = (int64_t)blockIdx.x * chunk;
    const int64_t tend = min(t + chunk, g.tiles);
    if (t >= tend)
        return;
    TileTaps<DT, K> taps;
    V bias = V(0), v_th;
    if constexpr (kF)
        v_th = a.v_th;
    else
        v_th = a.v_th_q;
    int cur = -1, cur_W = -1, top = 0;
    const int ch = q / g.ncls, r0 = q - ch * g.ncls;  // (ch 0 when a row has more classes than lanes)
    const int N = (int)divide(a.M, (int64_t)g.S * g.C);
    Part part{};
    Cursor tl(g, t);
    for (; t < tend; ++t, tl.next(g, N)) {
        if (tl.p != cur) {
            cur = tl.p;
            const int c = g.by_channel ? cur : (int)divide((int64_t)cur * g.G + min(row, tl.rows - 1), g.S);
            taps.load(a.sign, a.shift, c, a.shift_lo, a.shift_hi);
            if constexpr (kF) {
                const float b = ((const float*)a.bias)[c];
                bias = b == 0.0f ? 0.0f : b;  // a zero bias is added as +0
            } else {
                bias = ((const int32_t*)a.bias)[c];
            }
        }
        const int W = min(g.seg, g.T - tl.t0);        // steps of the tile
        if (W != cur_W) {  // (the same for every tile but a column's last)
            cur_W = W;
            top = tile_chunk(g, W);
            part = part_of(g, W, r0, ch, top);
        }
        const int before = min(g.span, tl.t0);        // history staged before them
        const int count = g.nseg == 1 ? tl.rows * g.T : before + W;
        const int64_t e0 = tl.col0 * g.T + tl.t0;
        ExactCheck chk;
        int off, off2;
        const bool check = kF && a.x_exact == 0;
        if (check)
            stage<DT, false, true, 4>(g, a.x, e0 - before, count, nullptr, 0, 0, total, a.vec_x, xi, nullptr, chk,
                                      off, off2);
        else
            stage<DT, false, false, 4>(g, a.x, e0 - before, count, nullptr, 0, 0, total, a.vec_x, xi, nullptr, chk,
                                       off, off2);
        bool slow = false;
        if constexpr (kF)
            slow = check && (a.fast_hi < INFINITY || __builtin_amdgcn_ballot_w64(chk.inexact(a.fast_lo)) != 0);
        wave_sync();
        const int ooff = WANT_H ? (a.vec_h ? (int)(e0 & 3) : 0) : a.vec_s ? (int)(e0 & 15) : 0;
        // byte addresses of the row's first step in the images
        const int xrow = (off + before + row * g.xs) * es, orow = g.lds_x + (ooff + row * g.os) * os;
        auto walk = [&](auto exact, const Part& pt) __attribute__((always_inline)) {
            constexpr bool EX = decltype(exact)::value;
            const int hist = tl.t0 > 0 ? K : pt.j0;  // steps of the class before the chunk (at least k, or all)
            const int at = pt.r + pt.j0 * g.d;
            int xa = xrow + at * es, oa = orow + at * os;
            V ring[K];  // step s of the chunk at slot s mod k
#pragma unroll
            for (int b = 0; b < K; ++b)
                ring[b] = V(0);
            if (g.m > 1 || tl.t0 > 0) {
#pragma unroll
                for (int b = 1; b < K; ++b) {
                    const V v = IO::get(*(const E*)(lds + (b <= hist ? xa - b * xstep : xa)));
                    ring[K - b] = b <= hist ? v : V(0);
                }
            }
            walk_steps<K>(top, pt.j1 - pt.j0, [&](auto uc) __attribute__((always_inline)) {
                constexpr int u = decltype(uc)::value;
                ring[u] = IO::get(*(const E*)(lds + xa));
                V acc;
                if constexpr (kF) {
                    acc = ring[(u + 1) % K] * taps.w[0];
#pragma unroll
                    for (int i = 1; i < K; ++i)
                        acc = taps.template add<EX>(acc, ring[(u + 1 + i) % K], i);
                } else {
                    acc = taps.start();
#pragma unroll
                    for (int i = 0; i < K; ++i)
                        acc = taps.template add<EX>(acc, ring[(u + 1 + i) % K], i);
                }
                const V h = acc + bias;
                if constexpr (WANT_H)
                    *(V*)(lds + oa) = h;
                else
                    lds[oa] = h >= v_th ? 1 : 0;
                xa += xstep;
                oa += g.d * os;
            });
        };
        if (mine && row < tl.rows) {
            Part pt = part;
            for (int r = r0;;) {
                if (kF && slow)
                    walk(std::true_type{}, pt);
                else
                    walk(std::false_type{}, pt);
                if (g.ncls <= 64 || (r += 64) >= g.ncls)
                    break;
                pt = part_of(g, W, r, 0, top);
            }
        }
        wave_sync();
        const int out = g.nseg == 1 ? count : W;
        if constexpr (WANT_H)
            unstage_h<V>(g, (const V*)oi, ooff, out, v_th, (V*)a.h_out, a.spikes, e0, a.vec_h);
        else
            unstage<uint8_t, uint8_t>(g, (const uint8_t*)oi, ooff, out, g.os, a.spikes, e0, a.vec_s);
        wave_sync();  // every read of the images before the next tile's writes
    }
}

template <typename W> __device__ __forceinline__ W lanes_sum(W v)
{
#pragma unroll
    for (int j = 1; j < 64; j <<= 1) {
        if constexpr (std::is_same_v<W, double>) {
            v += __shfl_xor(v, j, 64);
        } else {
            const int lo = __shfl_xor((int)(uint32_t)v, j, 64);
            const int hi = __shfl_xor((int)(uint32_t)((uint64_t)v >> 32), j, 64);
            v += (int64_t)(((uint64_t)(uint32_t)hi << 32) | (uint32_t)lo);
        }
    }
    return v;
}

template <int DT, int K>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(K <= 8 ? 4 : K <= 16 ? 3 : 2))) void tile_bwd_kernel(
    TlBwdArgs a, TileGeom g)
{
    using IO = TileIO<DT>;
    using V = typename IO::V;
    using E = typename IO::E;
    using W = typename IO::W;
    constexpr bool kF = DT != MFPSN_Q8_8;
    constexpr int es = (int)sizeof(E);
    extern __shared__ __attribute__((aligned(16))) char lds[];
    char* xi = lds;
    char* di = lds + g.lds_x;
    const int xstep = g.d * es, dstep = g.d * 4;
    const int lane = (int)threadIdx.x;
    const int row = min(lane / g.Q, g.G - 1), q = lane - row * g.Q;
    const bool mine = q < g.ncls * g.m && lane < g.G * g.Q;
    const int64_t total = a.M * a.T;
    int64_t t = (int64_t)blockIdx.x * a.chunk;
    const int64_t tend = min(t + a.chunk, g.tiles);
    if (t >= tend)
        return;
    Surrogate sg;
    sg.init(a.sg, a.alpha);
    TileTaps<DT, K> taps;
    V bias = V(0);
    W gw[K], gb = W(0);
#pragma unroll
    for (int i = 0; i < K; ++i)
        gw[i] = W(0);
    int cur = -1, cur_rows = 0, cur_own = -1, cur_win = -1, top1 = 0, top2 = 0;
    int64_t cur_z = 0;  // the first tile of group cur this wave meets
    const int ch = q / g.ncls, r0 = q - ch * g.ncls;  // (ch 0 when a row has more classes than lanes)
    const int N = (int)divide(a.M, (int64_t)g.S * g.C);
    Part part1{}, part2{};
    // the sums of the lanes of each channel of group `cur`, to its slots
    auto flush = [&]() __attribute__((always_inline)) {
        W* slot = (W*)a.part + tile_slot(g, blockIdx.x, cur_z, cur) * (K + 1);
        if (g.by_channel) {
#pragma unroll
            for (int i = 0; i <= K; ++i) {
                const W v = lanes_sum(i < K ? gw[i < K ? i : 0] : gb);
                if (lane == 0)
                    slot[i] = v;
            }
        } else {
            // lane ch adds the lanes of the rows of channel c0 + ch
            const int64_t j0 = (int64_t)cur * g.G;
            const int c0 = (int)(j0 / g.S);
            const int last = (int)((j0 + cur_rows - 1) / g.S) - c0;
            const int lo = (int)max((int64_t)0, (int64_t)(c0 + lane) * g.S - j0);
            const int hi = (int)min((int64_t)cur_rows, (int64_t)(c0 + lane + 1) * g.S - j0);
            W* red = (W*)lds;
            for (int i = 0; i <= K; ++i) {
                W mineW = gb;
#pragma unroll
                for (int j = 0; j < K; ++j)
                    mineW = i == j ? gw[j] : mineW;
                red[lane] = mineW;
                wave_sync();
                if (lane <= last) {
                    W v = W(0);
                    for (int l = lo * g.Q; l < hi * g.Q; ++l)
                        v += red[l];
                    slot[lane * (K + 1) + i] = v;
                }
                wave_sync();
            }
        }
#pragma unroll
        for (int i = 0; i < K; ++i)
            gw[i] = W(0);
        gb = W(0);
    };
    Cursor tl(g, t);
    for (; t < tend; ++t, tl.next(g, N)) {
        if (tl.p != cur) {
            if (cur >= 0)
                flush();
            cur = tl.p;
            cur_z = tl.z(g);
            cur_rows = tl.rows;
            const int c = g.by_channel ? cur : (int)divide((int64_t)cur * g.G + min(row, tl.rows - 1), g.S);
            taps.load(a.sign, a.shift, c, a.shift_lo, a.shift_hi);
            if constexpr (kF) {
                const float b = ((const float*)a.bias)[c];
                bias = b == 0.0f ? 0.0f : b;
            } else {
                bias = ((const int32_t*)a.bias)[c];
            }
        }
        const int own = min(g.seg, g.T - tl.t0);               // steps of the tile
        const int win = min(own + g.span, g.T - tl.t0);        // and those after them its grad_x needs
        const int before = min(g.span, tl.t0);
        const bool whole = g.nseg == 1;
        if (own != cur_own || win != cur_win) {  // (the same for every tile but a column's last)
            cur_own = own;
            cur_win = win;
            top1 = tile_chunk(g, win);
            top2 = tile_chunk(g, own);
            part1 = part_of(g, win, r0, ch, top1);
            part2 = part_of(g, own, r0, ch, top2);
        }
        const int64_t e0 = tl.col0 * g.T + tl.t0;
        ExactCheck chk;
        int xoff, doff;
        const bool check = kF && a.x_exact == 0;
        const int count = whole ? tl.rows * g.T : win;
        if (check)
            stage<DT, true, true, 4>(g, a.x, e0 - before, before + count, a.g, e0, count, total, a.vec_x, xi, di, chk,
                                     xoff, doff);
        else
            stage<DT, true, false, 4>(g, a.x, e0 - before, before + count, a.g, e0, count, total, a.vec_x, xi, di, chk,
                                      xoff, doff);
        bool slow = false;
        if constexpr (kF)
            slow = check && (a.fast_hi < INFINITY || __builtin_amdgcn_ballot_w64(chk.inexact(a.fast_lo)) != 0);
        wave_sync();
        // byte addresses of the row's first step in the images
        const int xrow = (xoff + before + row * g.xs) * es, drow = g.lds_x + (doff + row * g.os) * 4;
        const bool live = mine && row < tl.rows;

        // H and dH over the window, grad_w and grad_b over the tile's steps
        ExactCheck chk_d;
        auto walk1 = [&](auto exact, const Part& pt) __attribute__((always_inline)) {
            constexpr bool EX = decltype(exact)::value;
            const int hist = tl.t0 > 0 ? K : pt.j0;
            const int at = pt.r + pt.j0 * g.d;
            int xa = xrow + at * es, da = drow + at * 4;
            const int dend = drow + own * 4;  // the tile's own steps lie below
            V ring[K];
            W xd[kF ? K : 1];
#pragma unroll
            for (int b = 0; b < K; ++b) {
                ring[b] = V(0);
                if constexpr (kF)
                    xd[b] = W(0);
            }
            if (g.m > 1 || tl.t0 > 0) {
#pragma unroll
                for (int b = 1; b < K; ++b) {
                    const V v = IO::get(*(const E*)(lds + (b <= hist ? xa - b * xstep : xa)));
                    ring[K - b] = b <= hist ? v : V(0);
                    if constexpr (kF)
                        xd[K - b] = (W)ring[K - b];
                }
            }
            walk_steps<K>(top1, pt.j1 - pt.j0, [&](auto uc) __attribute__((always_inline)) {
                constexpr int u = decltype(uc)::value;
                ring[u] = IO::get(*(const E*)(lds + xa));
                V* dp = (V*)(lds + da);
                const V gv = *dp;
                if constexpr (kF)
                    xd[u] = (W)ring[u];
                V acc;
                if constexpr (kF) {
                    acc = ring[(u + 1) % K] * taps.w[0];
#pragma unroll
                    for (int i = 1; i < K; ++i)
                        acc = taps.template add<EX>(acc, ring[(u + 1 + i) % K], i);
                } else {
                    acc = taps.start();
#pragma unroll
                    for (int i = 0; i < K; ++i)
                        acc = taps.template add<EX>(acc, ring[(u + 1 + i) % K], i);
                }
                const V dh = delta_h(gv, sg_factor(sg, acc + bias, a.v_th, a.v_th_q));
                *dp = dh;
                if constexpr (kF)
                    chk_d.see(dh);
                // (a history step after the tile adds zeros: its products are
                // the next tile's)
                V dw = dh;
                if (!whole) {
                    asm volatile("" : "+v"(dw));  // (a branch, not a select on every step)
                    dw = da < dend ? dw : V(0);
                }
                if constexpr (kF) {
                    const W dd = (W)dw;
#pragma unroll
                    for (int i = 0; i < K; ++i)
                        gw[i] = __builtin_fma(xd[(u + 1 + i) % K], dd, gw[i]);
                    gb += dd;
                } else {
#pragma unroll
                    for (int i = 0; i < K; ++i) {
                        gw[i] += (int64_t)ring[(u + 1 + i) % K] * (int64_t)dw;
                        pin(gw[i]);
                    }
                    gb += dw;
                }
                xa += xstep;
                da += dstep;
                __builtin_amdgcn_sched_barrier(0);
            });
        };
        if (live) {
            Part pt = part1;
            for (int r = r0;;) {
                if (kF && slow)
                    walk1(std::true_type{}, pt);
                else
                    walk1(std::false_type{}, pt);
                if (g.ncls <= 64 || (r += 64) >= g.ncls)
                    break;
                pt = part_of(g, win, r, 0, top1);
            }
        }
        wave_sync();
        bool slow_d = false;
        if constexpr (kF)
            slow_d = a.fast_hi < INFINITY || __builtin_amdgcn_ballot_w64(chk_d.inexact(a.fast_lo)) != 0;

        // grad_x over the tile's steps, from the last down
        auto walk2 = [&](auto exact, const Part& pt, int Lw) __attribute__((always_inline)) {
            constexpr bool EX = decltype(exact)::value;
            const int after = Lw - pt.j1;  // steps of the class after the chunk that have a dH
            int da = drow + (pt.r + (pt.j1 - 1) * g.d) * 4;
            V ring[K];  // dH of step s of the walk at slot s mod k
#pragma unroll
            for (int b = 0; b < K; ++b)
                ring[b] = V(0);
            if (g.m > 1 || !whole) {
#pragma unroll
                for (int b = 1; b < K; ++b) {
                    const V v = *(const V*)(lds + (b <= after ? da + b * dstep : da));
                    ring[K - b] = b <= after ? v : V(0);
                }
            }
            walk_steps<K>(top2, pt.j1 - pt.j0, [&](auto uc) __attribute__((always_inline)) {
                constexpr int u = decltype(uc)::value;
                V* dp = (V*)(lds + da);
                ring[u] = *dp;
                // dH of step j + (k-1-i) sits k-1-i steps back in the walk
                V acc = taps.start();
#pragma unroll
                for (int i = 0; i < K; ++i)
                    acc = taps.template add<EX>(acc, ring[(u + 1 + i) % K], i);
                *dp = acc;
                da -= dstep;
            });
        };
        if (live) {
            // (a row with more classes than lanes walks them one after
            // another: the classes are independent)
            Part pt = part2;
            int Lw = part1.L;
            for (int r = r0;;) {
                if (kF && slow_d)
                    walk2(std::true_type{}, pt, Lw);
                else
                    walk2(std::false_type{}, pt, Lw);
                if (g.ncls <= 64 || (r += 64) >= g.ncls)
                    break;
                pt = part_of(g, own, r, 0, top2);
                Lw = part_of(g, win, r, 0, top1).L;
            }
        }
        wave_sync();
        const int out = whole ? count : own;
        if constexpr (DT == MFPSN_BF16)
            unstage<float, uint16_t>(g, (const float*)di, doff, out, g.os, (uint16_t*)a.grad_x, e0, a.vec_o);
        else
            unstage<V, V>(g, (const V*)di, doff, out, g.os, (V*)a.grad_x, e0, a.vec_o);
        wave_sync();  // every read of the images before the next tile's writes
    }
    flush();
}

// grad_w and grad_b from the slots of partial sums: one block per channel.
// The k + 1 sums of a slot are neighbours, so a wave reads 64 / (k + 1) slots
// at once (lane = slot, sum) and the waves take turns; then each wave adds
// its lanes' slots and the waves' sums are added, all in a fixed order: the
// same bits on every call.
constexpr int kFinWaves = 16;

template <typename W>
__global__ __launch_bounds__(64 * kFinWaves) void tile_fin_kernel(const W* part, TileGeom g, int64_t chunk, int32_t k1,
                                                                  void* grad_w, void* grad_b)
{
    const int c = blockIdx.x, lane = (int)threadIdx.x & 63, v = (int)threadIdx.x >> 6;
    const int per = 64 / k1, sub = lane / k1, i = lane - sub * k1, hop = per * kFinWaves;
    int p0 = c, p1 = c;
    if (!g.by_channel) {
        p0 = (int)((int64_t)c * g.S / g.G);
        p1 = (int)(((int64_t)c * g.S + g.S - 1) / g.G);
    }
    W s = W(0);
    for (int p = p0; p <= p1 && sub < per; ++p) {
        const int ch = g.by_channel ? 0 : c - (int)((int64_t)p * g.G / g.S);
        const int64_t first = (int64_t)p * g.Z / chunk, last = ((int64_t)(p + 1) * g.Z - 1) / chunk;
        auto slot = [&](int64_t w) {
            const int64_t z = w * chunk - (int64_t)p * g.Z;
            return part[(tile_slot(g, w, z > 0 ? z : 0, p) + ch) * k1 + i];
        };
        int64_t w = first + v * per + sub;
        for (; w + 7 * hop <= last; w += 8 * hop) {
            W t[8];
#pragma unroll
            for (int u = 0; u < 8; ++u)
                t[u] = slot(w + u * hop);
#pragma unroll
            for (int u = 0; u < 8; ++u)
                s += t[u];
        }
        for (; w <= last; w += hop)
            s += slot(w);
    }
    __shared__ W red[kFinWaves][64];
    red[v][lane] = s;
    wave_sync();
    for (int q = 1; q < per && lane < k1; ++q)
        s += red[v][q * k1 + lane];
    wave_sync();
    red[v][lane] = s;
    __syncthreads();
    if (v != 0 || lane >= k1)
        return;
    for (int q = 1; q < kFinWaves; ++q)
        s += red[q][lane];
    using O = std::conditional_t<std::is_same_v<W, double>, float, int64_t>;
    if (lane < k1 - 1)
        ((O*)grad_w)[(int64_t)c * (k1 - 1) + lane] = (O)s;
    else
        ((O*)grad_b)[c] = (O)s;
}

// Waves of `kern` with `lds` bytes each that fit on the current device at
// once: by registers (asked once per kernel and device: blocks per CU and CUs
// in one word, so that threads making a kernel's first calls see both or
// neither; 0: not asked yet) and by LDS
using WaveCache = std::atomic<uint32_t>[64];
template <typename Kern> int64_t resident_waves(Kern kern, WaveCache& cache, int lds)
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0)
        dev = 0;
    uint32_t known = dev < 64 ? cache[dev].load(std::memory_order_relaxed) : 0;
    if (known == 0) {
        int per = 0, cus = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per, kern, 64, 0) != hipSuccess || per < 1)
            per = 1;
        if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1)
            cus = 1;
        known = (uint32_t)per << 16 | (uint32_t)(cus < 0xFFFF ? cus : 0xFFFF);
        if (dev < 64)
            cache[dev].store(known, std::memory_order_relaxed);
    }
    const int fit = 163840 / ((lds + 1279) / 1280 * 1280), per = (int)(known >> 16);
    return (int64_t)(per < fit ? per : fit) * (known & 0xFFFFu);
}

template <int DT, int K, bool WANT_H> hipError_t fwd_tiles(const TlArgs& a, const TileGeom& g, hipStream_t st)
{
    static WaveCache cache;
    auto kern = tile_fwd_kernel<DT, K, WANT_H>;
    const int64_t waves = tile_waves(g, resident_waves(kern, cache, g.lds), -1);
    if (waves < 1)
        return hipErrorInvalidValue;
    const int64_t chunk = (g.tiles + waves - 1) / waves;
    const unsigned blocks = (unsigned)((g.tiles + chunk - 1) / chunk);
    hipLaunchKernelGGL(kern, dim3(blocks), dim3(64), (size_t)g.lds, st, a, g, chunk);
    return hipGetLastError();
}

template <int DT, int K> hipError_t bwd_tiles(TlBwdArgs& a, const TileGeom& g, int64_t slots, hipStream_t st)
{
    static WaveCache cache;
    auto kern = tile_bwd_kernel<DT, K>;
    const int64_t waves = tile_waves(g, resident_waves(kern, cache, g.lds), slots);
    if (waves < 1)
        return hipErrorInvalidValue;
    a.chunk = (g.tiles + waves - 1) / waves;
    const unsigned blocks = (unsigned)((g.tiles + a.chunk - 1) / a.chunk);
    hipLaunchKernelGGL(kern, dim3(blocks), dim3(64), (size_t)g.lds, st, a, g);
    return hipGetLastError();
}

template <int DT, int LO, int... Ks>
hipError_t fwd_range(const TlArgs& a, const TileGeom& g, hipStream_t st, std::integer_sequence<int, Ks...>)
{
    hipError_t e = hipErrorInvalidValue;
    if (a.h_out != nullptr)
        (void)((a.k == LO + Ks ? (e = fwd_tiles<DT, LO + Ks, true>(a, g, st), true) : false) || ...);
    else
        (void)((a.k == LO + Ks ? (e = fwd_tiles<DT, LO + Ks, false>(a, g, st), true) : false) || ...);
    return e;
}
template <int DT, int LO, int... Ks>
hipError_t bwd_range(TlBwdArgs& a, const TileGeom& g, int64_t slots, hipStream_t st, std::integer_sequence<int, Ks...>)
{
    hipError_t e = hipErrorInvalidValue;
    (void)((a.k == LO + Ks ? (e = bwd_tiles<DT, LO + Ks>(a, g, slots, st), true) : false) || ...);
    return e;
}

}  // namespace

// Compiled once per storage type and range of orders (MFPSN_TILE_DTYPE,
// MFPSN_TILE_KLO .. MFPSN_TILE_KHI); the unit without them holds the dispatch.
#if defined(MFPSN_TILE_DTYPE)
using TileKs = std::make_integer_sequence<int, MFPSN_TILE_KHI - MFPSN_TILE_KLO + 1>;
template <>
hipError_t tile_forward<MFPSN_TILE_DTYPE, MFPSN_TILE_KLO>(const TlArgs& a, const TileGeom& g, hipStream_t st)
{
    return fwd_range<MFPSN_TILE_DTYPE, MFPSN_TILE_KLO>(a, g, st, TileKs{});
}
template <>
hipError_t tile_backward<MFPSN_TILE_DTYPE, MFPSN_TILE_KLO>(TlBwdArgs& a, const TileGeom& g, int64_t slots,
                                                           hipStream_t st)
{
    return bwd_range<MFPSN_TILE_DTYPE, MFPSN_TILE_KLO>(a, g, slots, st, TileKs{});
}
#else
namespace {
template <int DT> hipError_t fwd_dtype(const TlArgs& a, const TileGeom& g, hipStream_t st)
{
    if (a.k <= kTileKs[1] - 1)
        return tile_forward<DT, kTileKs[0]>(a, g, st);
    if (a.k <= kTileKs[2] - 1)
        return tile_forward<DT, kTileKs[1]>(a, g, st);
    if (a.k <= kTileKs[3] - 1)
        return tile_forward<DT, kTileKs[2]>(a, g, st);
    return tile_forward<DT, kTileKs[3]>(a, g, st);
}
template <int DT> hipError_t bwd_dtype(TlBwdArgs& a, const TileGeom& g, int64_t slots, hipStream_t st)
{
    if (a.k <= kTileKs[1] - 1)
        return tile_backward<DT, kTileKs[0]>(a, g, slots, st);
    if (a.k <= kTileKs[2] - 1)
        return tile_backward<DT, kTileKs[1]>(a, g, slots, st);
    if (a.k <= kTileKs[3] - 1)
        return tile_backward<DT, kTileKs[2]>(a, g, slots, st);
    return tile_backward<DT, kTileKs[3]>(a, g, slots, st);
}
}  // namespace

hipError_t launch_forward_tiles(const TlArgs& a, const TileGeom& g, int dtype, hipStream_t st)
{
    switch (dtype) {
    case MFPSN_F32: return fwd_dtype<MFPSN_F32>(a, g, st);
    case MFPSN_BF16: return fwd_dtype<MFPSN_BF16>(a, g, st);
    default: return fwd_dtype<MFPSN_Q8_8>(a, g, st);
    }
}

hipError_t launch_backward_tiles(TlBwdArgs& a, const TileGeom& g, int64_t slots, int dtype, void* grad_w,
                                 void* grad_b, hipStream_t st)
{
    hipError_t e;
    switch (dtype) {
    case MFPSN_F32: e = bwd_dtype<MFPSN_F32>(a, g, slots, st); break;
    case MFPSN_BF16: e = bwd_dtype<MFPSN_BF16>(a, g, slots, st); break;
    default: e = bwd_dtype<MFPSN_Q8_8>(a, g, slots, st); break;
    }
    if (e != hipSuccess)
        return e;
    const dim3 grid((unsigned)a.C), block(64 * kFinWaves);
    if (dtype == MFPSN_Q8_8)
        hipLaunchKernelGGL(tile_fin_kernel<int64_t>, grid, block, 0, st, (const int64_t*)a.part, g, a.chunk,
                           a.k + 1, grad_w, grad_b);
    else
        hipLaunchKernelGGL(tile_fin_kernel<double>, grid, block, 0, st, (const double*)a.part, g, a.chunk,
                           a.k + 1, grad_w, grad_b);
    return hipGetLastError();
}
#endif

}  // namespace mfpsn
