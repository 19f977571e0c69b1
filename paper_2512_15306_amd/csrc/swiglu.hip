// SwiGLU with the extra outputs the FP8 pipeline wants from a non-linearity (paper Section 3,
// kernel-fusion paragraph: every non-linearity also returns the absmax of its result, so the FP8
// conversion of the next matmul's input needs no reduction pass; Section 3 "Activation checkpointing":
// when the absmax is already known, as in recomputation during backward, the conversion itself is
// fused into the non-linearity).
//
//   GU [M, 2I] BF16: columns [0, I) gate g, columns [I, 2I) up u;   h[m,i] = bf16( silu(g) * u )
//   backward: dGU[m, i] = bf16( dh u sg (1 + g (1 - sg)) ),  dGU[m, I+i] = bf16( dh g sg ),  sg = sigma(g)
//
// HBM-bound (forward 4 B read + 2 B written per element of h, or + 1 B + 1 B when FP8 bytes replace
// h; backward 6 B read + 4 B written), with the arithmetic not far behind (sigmoid_f32_normal).  A lane owns a patch of
// PR rows x 8 columns, the shape of the quantize kernels, so the FP8 mode reuses their transposes: 16-byte loads of g and
// u, arithmetic in binary32, hardware RNE conversion to BF16, packed 16-bit integer absmax on the
// rounded bits, one partial absmax per workgroup (a second kernel reduces them; no atomics).
//
// The arithmetic is fixed operation by operation (IEEE binary32, nothing contracted beyond the
// fused multiply-adds written out) so that the stored bits can be reproduced anywhere:
//   a = -min(max(g,-100),86); n = rint(a*LOG2E); r = fma(n,-LN2_HI,a); r = fma(n,-LN2_LO,r);
//   p = Horner of 1 + r + r^2/2 + ... + r^6/720; e = p * 2^n; sg = 1 / (1 + e); h = (g*sg)*u.
#include <stdlib.h>

#include "llmq_device.h"
#include "llmq_kernels.h"

#pragma clang fp contract(off)

namespace llmq {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float v2f __attribute__((ext_vector_type(2)));

constexpr int kSwThreads = 256;
constexpr int kSwLanesR = 8;                                     // lanes stacked along rows
constexpr int kSwBlockCols = 8 * (kWave / kSwLanesR) * (kSwThreads / kWave);    // 256 columns per workgroup
constexpr int kSwEdgeMaxBlocks = 1024;

__device__ inline float sigmoid_f32(float g) {
    const float a = -__builtin_fminf(__builtin_fmaxf(g, -100.0f), 86.0f);
    const float n = __builtin_rintf(a * 0x1.715476p+0f);
    float r = __builtin_fmaf(n, -0x1.62e430p-1f, a);
    r = __builtin_fmaf(n, 0x1.05c610p-29f, r);
    float p = 0x1.6c16c2p-10f;
    p = __builtin_fmaf(p, r, 0x1.111112p-7f);
    p = __builtin_fmaf(p, r, 0x1.555556p-5f);
    p = __builtin_fmaf(p, r, 0x1.555556p-3f);
    p = __builtin_fmaf(p, r, 0.5f);
    p = __builtin_fmaf(p, r, 1.0f);
    p = __builtin_fmaf(p, r, 1.0f);
    const float e = __builtin_ldexpf(p, (int)n);
    const float d = 1.0f + e;
    return 1.0f / d;                                    // correctly rounded division
}

// The same bits for g >= -86 (finite) in two thirds of the instructions: the arithmetic, not the memory, bounded these
// kernels.  The lower clamp does nothing there, and 1 + e lies in [1, 2^125], where one Newton step on the hardware's
// reciprocal (v_rcp_f32, off by one unit at most) is the correctly rounded quotient: compared with the division for every
// binary32 in [1, 2^126).  The division's scaling and fix-up steps are for operands that do not occur.  8192 x 18944: forward
// 194 -> 174 us (5.3 TB/s), forward to FP8 222 -> 183 (5.1), backward 292 -> 287 (5.4).
__device__ inline float sigmoid_f32_normal(float g) {
    const float a = -__builtin_fminf(g, 86.0f);
    const float n = __builtin_rintf(a * 0x1.715476p+0f);
    float r = __builtin_fmaf(n, -0x1.62e430p-1f, a);
    r = __builtin_fmaf(n, 0x1.05c610p-29f, r);
    float p = 0x1.6c16c2p-10f;
    p = __builtin_fmaf(p, r, 0x1.111112p-7f);
    p = __builtin_fmaf(p, r, 0x1.555556p-5f);
    p = __builtin_fmaf(p, r, 0x1.555556p-3f);
    p = __builtin_fmaf(p, r, 0.5f);
    p = __builtin_fmaf(p, r, 1.0f);
    p = __builtin_fmaf(p, r, 1.0f);
    const float d = 1.0f + __builtin_ldexpf(p, (int)n);
    const float y = __builtin_amdgcn_rcpf(d);
    return __builtin_fmaf(__builtin_fmaf(-d, y, 1.0f), y, y);
}

// Whether all eight gates are >= -86 (or NaN, whose results are NaN either way): as unsigned numbers, the BF16 patterns
// of smaller ones are those above that of -86.
__device__ inline bool gates_normal(const v4u& g) {
    const unsigned m = pk_max_u16(pk_max_u16(g[0], g[1]), pk_max_u16(g[2], g[3]));
    return (m & 0xFFFFu) <= 0xC2ACu && (m >> 16) <= 0xC2ACu;
}

template <bool NORMAL>
__device__ inline float swiglu_f32(float g, float u) {
    const float silu = g * (NORMAL ? sigmoid_f32_normal(g) : sigmoid_f32(g));
    return silu * u;
}

__device__ inline unsigned pack_bf16(float lo, float hi) {
    v2f v = {lo, hi};
    return __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf16x2));   // RNE, low half = first
}

__device__ inline float bf16_lo(unsigned w) { return __uint_as_float(w << 16); }
__device__ inline float bf16_hi(unsigned w) { return __uint_as_float(w & 0xFFFF0000u); }

// Eight elements: one 16-byte vector of g and of u -> one 16-byte vector of h.
template <bool NORMAL>
__device__ __forceinline__ v4u swiglu8_as(const v4u& g, const v4u& u) {
    v4u o;
#pragma unroll
    for (int j = 0; j < 4; ++j)
        o[j] = pack_bf16(swiglu_f32<NORMAL>(bf16_lo(g[j]), bf16_lo(u[j])), swiglu_f32<NORMAL>(bf16_hi(g[j]), bf16_hi(u[j])));
    return o;
}
__device__ __attribute__((noinline)) v4u swiglu8_rare(v4u g, v4u u) { return swiglu8_as<false>(g, u); }
// CALL_RARE: the rare half as a call instead of in the kernel's code, of which it would be half.  Forward with h, aligned shapes, in the code / called:
// 1536 x 1408 8.8 / 8.7 us, 8192 x 256 8.6 / 8.3, 1024 x 3072 9.4 / 9.1, 1.5 % on average from half a million to 8 million elements and nothing
// elsewhere; codes without the transposed copy 4096 x 9216 39.3 / 36.8, 8960 x 4992 45.0 / 42.0, 8704 x 4224 39.2 / 37.5, on average 0.5 % above 16 million elements; in the guarded kernels, whose patches are loaded between branches, the call costs 1 %.
template <bool CALL_RARE = false>
__device__ inline v4u swiglu8(const v4u& g, const v4u& u) {
    if (__builtin_expect(gates_normal(g), 1)) return swiglu8_as<true>(g, u);
    if constexpr (CALL_RARE) return swiglu8_rare(g, u);
    return swiglu8_as<false>(g, u);
}

template <bool NORMAL>
__device__ inline void swiglu_bwd_f32(float d, float g, float u, float& dg, float& du) {
    const float sg = NORMAL ? sigmoid_f32_normal(g) : sigmoid_f32(g);
    const float silu = g * sg;
    du = d * silu;
    const float one_minus = 1.0f - sg;
    const float t = __builtin_fmaf(g, one_minus, 1.0f);
    float v = d * u;
    v = v * sg;
    dg = v * t;
}

// Eight elements of dh, g and u -> eight of the gate's and of the up branch's gradient (which may replace g and u)
template <bool NORMAL>
__device__ __forceinline__ void swiglu_bwd8_as(const v4u& d, const v4u& g, const v4u& u, v4u& og, v4u& ou) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        float dg0, du0, dg1, du1;
        swiglu_bwd_f32<NORMAL>(bf16_lo(d[j]), bf16_lo(g[j]), bf16_lo(u[j]), dg0, du0);
        swiglu_bwd_f32<NORMAL>(bf16_hi(d[j]), bf16_hi(g[j]), bf16_hi(u[j]), dg1, du1);
        og[j] = pack_bf16(dg0, dg1);
        ou[j] = pack_bf16(du0, du1);
    }
}
__device__ inline void swiglu_bwd8(const v4u& d, const v4u& g, const v4u& u, v4u& og, v4u& ou) {
    if (__builtin_expect(gates_normal(g), 1)) swiglu_bwd8_as<true>(d, g, u, og, ou);
    else swiglu_bwd8_as<false>(d, g, u, og, ou);
}

__device__ inline unsigned fold_max(unsigned m0, unsigned m1, unsigned m2, unsigned m3) {
    m0 = pk_max_mag(pk_max_mag(m0, m1), pk_max_mag(m2, m3));
    return (m0 & 0xFFFFu) > (m0 >> 16) ? (m0 & 0xFFFFu) : (m0 >> 16);
}

// Forward.  PR rows per lane.  Optional outputs: h (WRITE_H), a per-workgroup absmax (AMAX), FP8 codes with a given scale
// (QFMT >= 0).  M % PR == 0 and I % 8 == 0: a patch is all inside or all outside.
template <int PR, bool WRITE_H, bool AMAX, int QFMT, bool STREAM>
__global__ __launch_bounds__(kSwThreads) void swiglu_fwd_patch_kernel(
    const uint16_t* __restrict__ gu, int64_t M, int64_t I, uint16_t* __restrict__ h,
    unsigned* __restrict__ partial, const float* __restrict__ d_qscale, uint8_t* __restrict__ q, unsigned grid_cols) {
    __shared__ unsigned s_part[kSwThreads / kWave];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x / kWave;
    // consecutive workgroups walk along the columns (measured a few percent faster than down the rows)
    const unsigned brow = blockIdx.x / grid_cols, bcol = blockIdx.x % grid_cols;
    const int64_t r0 = (int64_t)brow * (PR * kSwLanesR) + (lane % kSwLanesR) * PR;
    const int64_t c0 = (int64_t)bcol * kSwBlockCols + wave * (8 * (kWave / kSwLanesR)) + (lane / kSwLanesR) * 8;
    unsigned mag = 0;
    if (r0 < M && c0 < I) {
        const uint16_t* src = gu + r0 * (2 * I) + c0;
        float s = 0.0f;
        if constexpr (QFMT >= 0) s = *d_qscale;
        unsigned m0 = 0, m1 = 0, m2 = 0, m3 = 0;
        v4u g[PR], u[PR], o[PR];
#pragma unroll
        for (int i = 0; i < PR; ++i) {
            g[i] = __builtin_nontemporal_load(reinterpret_cast<const v4u*>(src + (int64_t)i * 2 * I));
            u[i] = __builtin_nontemporal_load(reinterpret_cast<const v4u*>(src + (int64_t)i * 2 * I + I));
        }
#pragma unroll
        for (int i = 0; i < PR; ++i) o[i] = swiglu8<!STREAM>(g[i], u[i]);
        if constexpr (WRITE_H) {
            uint16_t* dst = h + r0 * I + c0;
#pragma unroll
            for (int i = 0; i < PR; ++i) store_hinted<STREAM>(o[i], reinterpret_cast<v4u*>(dst + (int64_t)i * I));
        }
        if constexpr (AMAX) {
#pragma unroll
            for (int i = 0; i < PR; ++i) {
                m0 = pk_max_mag(m0, o[i][0]);
                m1 = pk_max_mag(m1, o[i][1]);
                m2 = pk_max_mag(m2, o[i][2]);
                m3 = pk_max_mag(m3, o[i][3]);
            }
            mag = fold_max(m0, m1, m2, m3);
        }
        if constexpr (QFMT >= 0) {
            uint8_t* dq = q + r0 * I + c0;
#pragma unroll
            for (int i = 0; i < PR; ++i) {
                unsigned lo, hi;
                quantize8<QFMT>(o[i], s, lo, hi);
                store_hinted<STREAM>(v2u{lo, hi}, reinterpret_cast<v2u*>(dq + (int64_t)i * I));
            }
        }
    }
    if constexpr (AMAX) {
        mag = block_max_u32<kSwThreads>(mag, s_part);
        if (threadIdx.x == 0) partial[blockIdx.x] = mag;
    }
}

// FP8 codes in both layouts for tensors made of whole 128 x 128 tiles (every benchmark shape): the lane geometry
// and the LDS transpose of the quantize kernel's tile variant, so that all four streams (g, u, q, q_t) move in
// full 128-byte lines, and the transposed copy can be written in slabs.  Sixteen 16-byte loads in flight per lane.
// (8192 x 18944 in slabs on 128 x 256 tiles, 16 rows per lane in two groups: 187 us, now 174.)
template <bool WRITE_H, int QFMT, bool STREAM>
__global__ __launch_bounds__(kTileThreads) void swiglu_fwd_tile_kernel(
    const uint16_t* __restrict__ gu, int64_t I, uint16_t* __restrict__ h,
    const float* __restrict__ d_qscale, uint8_t* __restrict__ q, uint8_t* __restrict__ qt, unsigned grid_cols,
    int64_t qt_row_stride, int64_t qt_band_stride) {
    __shared__ __attribute__((aligned(16))) uint8_t s_t[kTileLdsBytes];
    const unsigned brow = blockIdx.x / grid_cols, bcol = blockIdx.x - brow * grid_cols;   // along the columns first
    int tr, tc;
    tile_patch_origin(tr, tc);
    const int64_t r0 = (int64_t)brow * kTileRows + tr, c0 = (int64_t)bcol * kTileCols + tc;
    const uint16_t* src = gu + r0 * (2 * I) + c0;
    const float s = *d_qscale;
    unsigned w[kPatchRows][2];
    v4u g[kPatchRows], u[kPatchRows], o[kPatchRows];
#pragma unroll
    for (int i = 0; i < kPatchRows; ++i) {
        g[i] = __builtin_nontemporal_load(reinterpret_cast<const v4u*>(src + (int64_t)i * 2 * I));
        u[i] = __builtin_nontemporal_load(reinterpret_cast<const v4u*>(src + (int64_t)i * 2 * I + I));
    }
#pragma unroll
    for (int i = 0; i < kPatchRows; ++i) o[i] = swiglu8(g[i], u[i]);
    if constexpr (WRITE_H) {
        uint16_t* dst = h + r0 * I + c0;
#pragma unroll
        for (int i = 0; i < kPatchRows; ++i) *reinterpret_cast<v4u*>(dst + (int64_t)i * I) = o[i];
    }
#pragma unroll
    for (int i = 0; i < kPatchRows; ++i) quantize8<QFMT>(o[i], s, w[i][0], w[i][1]);
    uint8_t* dq = q + r0 * I + c0;
#pragma unroll
    for (int i = 0; i < kPatchRows; ++i) store_hinted<STREAM>(v2u{w[i][0], w[i][1]}, reinterpret_cast<v2u*>(dq + (int64_t)i * I));
    tile_stage_transposed(w, tr, tc, s_t);
    __syncthreads();
    tile_write_transposed(s_t, qt + (int64_t)bcol * kTileCols * qt_row_stride + (int64_t)brow * qt_band_stride, qt_row_stride);
}

// Backward: dh [M, I], GU [M, 2I] -> dGU [M, 2I], one partial absmax per workgroup.  M % 4 == 0, I % 8 == 0.
template <bool STREAM>
__global__ __launch_bounds__(kSwThreads) void swiglu_bwd_patch_kernel(
    const uint16_t* __restrict__ dh, const uint16_t* __restrict__ gu, int64_t M, int64_t I,
    uint16_t* __restrict__ dgu, unsigned* __restrict__ partial, unsigned grid_cols) {
    constexpr int PR = 4;
    __shared__ unsigned s_part[kSwThreads / kWave];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x / kWave;
    const unsigned brow = blockIdx.x / grid_cols, bcol = blockIdx.x % grid_cols;
    const int64_t r0 = (int64_t)brow * (PR * kSwLanesR) + (lane % kSwLanesR) * PR;
    const int64_t c0 = (int64_t)bcol * kSwBlockCols + wave * (8 * (kWave / kSwLanesR)) + (lane / kSwLanesR) * 8;
    unsigned mag = 0;
    if (r0 < M && c0 < I) {
        const uint16_t* src = gu + r0 * (2 * I) + c0;
        const uint16_t* sd = dh + r0 * I + c0;
        v4u g[PR], u[PR], d[PR];
#pragma unroll
        for (int i = 0; i < PR; ++i) {
            g[i] = __builtin_nontemporal_load(reinterpret_cast<const v4u*>(src + (int64_t)i * 2 * I));
            u[i] = __builtin_nontemporal_load(reinterpret_cast<const v4u*>(src + (int64_t)i * 2 * I + I));
            d[i] = __builtin_nontemporal_load(reinterpret_cast<const v4u*>(sd + (int64_t)i * I));
        }
        unsigned m0 = 0, m1 = 0, m2 = 0, m3 = 0;
        uint16_t* dst = dgu + r0 * (2 * I) + c0;
#pragma unroll
        for (int i = 0; i < PR; ++i) {
            v4u og, ou;
            swiglu_bwd8(d[i], g[i], u[i], og, ou);
            store_hinted<STREAM>(og, reinterpret_cast<v4u*>(dst + (int64_t)i * 2 * I));
            store_hinted<STREAM>(ou, reinterpret_cast<v4u*>(dst + (int64_t)i * 2 * I + I));
            m0 = pk_max_mag(pk_max_mag(m0, og[0]), ou[0]);
            m1 = pk_max_mag(pk_max_mag(m1, og[1]), ou[1]);
            m2 = pk_max_mag(pk_max_mag(m2, og[2]), ou[2]);
            m3 = pk_max_mag(pk_max_mag(m3, og[3]), ou[3]);
        }
        mag = fold_max(m0, m1, m2, m3);
    }
    mag = block_max_u32<kSwThreads>(mag, s_part);
    if (threadIdx.x == 0) partial[blockIdx.x] = mag;
}

// Ragged shapes: guarded edges and vectors at any address (any I, any M).  Rows start at any even address, so a run
// of a row that a wave reads or writes touches one cache line more than it fills: a wave takes 4 rows x 512 columns, the
// 64 lanes side by side (1 KB runs), instead of the 64-column patches above.  The absmax-producing launches write one
// partial result per workgroup and their scratch holds few of them, so the workgroups walk over the waves' pieces.
constexpr int kSwEdgeRows = 4, kSwEdgeCols = 8 * kWave;
__device__ inline void swiglu_edge_origin(int64_t piece, unsigned col_pieces, int64_t& r0, int64_t& c0) {
    const int64_t g = piece / col_pieces;
    r0 = g * kSwEdgeRows;
    c0 = (piece - g * col_pieces) * kSwEdgeCols + (threadIdx.x & (kWave - 1)) * 8;
}
// Whether any lane's patch reaches over the tensor's edge (lanes beside the tensor have left): the same for all of a wave's lanes
__device__ inline bool swiglu_edge_guard(int64_t r0, int64_t c0, int64_t M, int64_t I) {
    return __ballot(M - r0 < kSwEdgeRows || I - c0 < 8) != 0;
}

__global__ __launch_bounds__(kSwThreads) void swiglu_fwd_edge_kernel(
    const uint16_t* __restrict__ gu, int64_t M, int64_t I, uint16_t* __restrict__ h, unsigned* __restrict__ partial,
    unsigned col_pieces, int64_t n_pieces) {
    constexpr int PR = kSwEdgeRows;
    __shared__ unsigned s_part[kSwThreads / kWave];
    unsigned m0 = 0, m1 = 0, m2 = 0, m3 = 0;
    constexpr int kWaves = kSwThreads / kWave;
    for (int64_t b = (int64_t)blockIdx.x * kWaves + threadIdx.x / kWave; b < n_pieces; b += (int64_t)gridDim.x * kWaves) {
        int64_t r0, c0;
        swiglu_edge_origin(b, col_pieces, r0, c0);
        if (c0 >= I) continue;
        const uint16_t* src = gu + r0 * (2 * I) + c0;
        v4u g[PR], u[PR], o[PR];
        with_guard(swiglu_edge_guard(r0, c0, M, I), [&](auto guard) {
            const int64_t rows_left = guard ? M - r0 : PR, cols_left = guard ? I - c0 : 8;
            load_patches_upto(c0, rows_left, cols_left, patch(g, src, 2 * I), patch(u, src + I, 2 * I));
#pragma unroll
            for (int i = 0; i < PR; ++i) {
                o[i] = swiglu8(g[i], u[i]);                 // zeros where nothing is: they do not raise the absmax
                m0 = pk_max_mag(m0, o[i][0]);
                m1 = pk_max_mag(m1, o[i][1]);
                m2 = pk_max_mag(m2, o[i][2]);
                m3 = pk_max_mag(m3, o[i][3]);
            }
            store_patch_upto(o, h + r0 * I + c0, I, rows_left, cols_left);
        });
    }
    const unsigned mag = block_max_u32<kSwThreads>(fold_max(m0, m1, m2, m3), s_part);
    if (threadIdx.x == 0) partial[blockIdx.x] = mag;
}

// FP8 codes with a given scale on the 64 x 128 tile, for ragged shapes and tensors of few tiles: h (if not NULL), q and
// the transposed copy (TRANSPOSE: plain, or slabs where the shape has them).
template <int QFMT, bool TRANSPOSE>
__global__ __launch_bounds__(kTileThreads) void swiglu_fwd_fp8_small_kernel(
    const uint16_t* __restrict__ gu, int64_t M, int64_t I, uint16_t* __restrict__ h,
    const float* __restrict__ d_qscale, uint8_t* __restrict__ q, uint8_t* __restrict__ qt, const SmallGrid grid,
    int64_t qt_row_stride, int64_t qt_band_stride) {
    __shared__ __attribute__((aligned(16))) uint8_t s_t[TRANSPOSE ? kSmallLdsBytes : 16];
    unsigned brow, bcol;
    if (!small_tile(grid, grid.first + blockIdx.x, brow, bcol)) return;
    int tr, tc;
    small_patch_origin(grid, tr, tc);
    const int64_t R0 = (int64_t)brow * kSmallRows, C0 = (int64_t)bcol * kSmallCols, r0 = R0 + tr, c0 = C0 + tc;
    const uint16_t* src = gu + r0 * (2 * I) + c0;
    with_guard(small_tile_guard(R0, C0, M, I), [&](auto guard) {
        const int64_t rows_left = guard ? M - r0 : kSmallPatch, cols_left = guard ? I - c0 : 8;
        v4u g[kSmallPatch], u[kSmallPatch];
        load_tile_patches_upto(c0, rows_left, cols_left, patch(g, src, 2 * I), patch(u, src + I, 2 * I));
        const float s = *d_qscale;
        unsigned w[kSmallPatch][2];
#pragma unroll
        for (int i = 0; i < kSmallPatch; ++i) {
            g[i] = swiglu8(g[i], u[i]);
            quantize8<QFMT>(g[i], s, w[i][0], w[i][1]);
        }
        if (h) store_patch_upto(g, h + r0 * I + c0, I, rows_left, cols_left);
        store_codes_upto(w, q + r0 * I + c0, I, rows_left, cols_left);
        if constexpr (TRANSPOSE) {
            small_stage_transposed(w, tr, tc, s_t);
            __syncthreads();
            small_write_transposed_upto(s_t, qt + C0 * qt_row_stride + (R0 / kTileRows) * qt_band_stride + R0 % kTileRows, qt_row_stride,
                                        guard ? M - R0 : kSmallRows, guard ? I - C0 : kSmallCols);
        }
    });
}

__global__ __launch_bounds__(kSwThreads) void swiglu_bwd_edge_kernel(
    const uint16_t* __restrict__ dh, const uint16_t* __restrict__ gu, int64_t M, int64_t I,
    uint16_t* __restrict__ dgu, unsigned* __restrict__ partial, unsigned col_pieces, int64_t n_pieces) {
    constexpr int PR = kSwEdgeRows;
    __shared__ unsigned s_part[kSwThreads / kWave];
    unsigned m0 = 0, m1 = 0, m2 = 0, m3 = 0;
    constexpr int kWaves = kSwThreads / kWave;
    for (int64_t b = (int64_t)blockIdx.x * kWaves + threadIdx.x / kWave; b < n_pieces; b += (int64_t)gridDim.x * kWaves) {
        int64_t r0, c0;
        swiglu_edge_origin(b, col_pieces, r0, c0);
        if (c0 >= I) continue;
        const uint16_t* src = gu + r0 * (2 * I) + c0;
        v4u g[PR], u[PR], d[PR];
        with_guard(swiglu_edge_guard(r0, c0, M, I), [&](auto guard) {
            const int64_t rows_left = guard ? M - r0 : PR, cols_left = guard ? I - c0 : 8;
            load_patches_upto(c0, rows_left, cols_left, patch(g, src, 2 * I), patch(u, src + I, 2 * I), patch(d, dh + r0 * I + c0, I));
#pragma unroll
            for (int i = 0; i < PR; ++i) {
                swiglu_bwd8(d[i], g[i], u[i], g[i], u[i]);
                m0 = pk_max_mag(pk_max_mag(m0, g[i][0]), u[i][0]);
                m1 = pk_max_mag(pk_max_mag(m1, g[i][1]), u[i][1]);
                m2 = pk_max_mag(pk_max_mag(m2, g[i][2]), u[i][2]);
                m3 = pk_max_mag(pk_max_mag(m3, g[i][3]), u[i][3]);
            }
            uint16_t* dst = dgu + r0 * (2 * I) + c0;
            store_patch_upto(g, dst, 2 * I, rows_left, cols_left);
            store_patch_upto(u, dst + I, 2 * I, rows_left, cols_left);
        });
    }
    const unsigned mag = block_max_u32<kSwThreads>(fold_max(m0, m1, m2, m3), s_part);
    if (threadIdx.x == 0) partial[blockIdx.x] = mag;
}

// FP8 codes in both layouts of narrow shapes of whole 16 x 8 patches; h may be NULL.
template <int QFMT>
__global__ __launch_bounds__(kSwThreads) void swiglu_fwd_fp8_narrow_kernel(
    const uint16_t* __restrict__ gu, int64_t M, int64_t I, uint16_t* __restrict__ h,
    const float* __restrict__ d_qscale, uint8_t* __restrict__ q, uint8_t* __restrict__ qt) {
    int tr, tc;
    narrow_patch_origin(tr, tc);
    const int64_t r0 = (int64_t)blockIdx.x * kNarrowRows + tr;
    if (r0 >= M || tc >= I) return;
    const uint16_t* src = gu + r0 * (2 * I) + tc;
    const float s = *d_qscale;
    constexpr int kGroup = 8;
    unsigned w[16][2];
#pragma unroll
    for (int i0 = 0; i0 < 16; i0 += kGroup) {
        v4u g[kGroup], u[kGroup];
#pragma unroll
        for (int i = 0; i < kGroup; ++i) {
            g[i] = __builtin_nontemporal_load(reinterpret_cast<const v4u*>(src + (int64_t)(i0 + i) * 2 * I));
            u[i] = __builtin_nontemporal_load(reinterpret_cast<const v4u*>(src + (int64_t)(i0 + i) * 2 * I + I));
        }
#pragma unroll
        for (int i = 0; i < kGroup; ++i) {
            const v4u o = swiglu8(g[i], u[i]);
            if (h) *reinterpret_cast<v4u*>(h + (r0 + i0 + i) * I + tc) = o;
            quantize8<QFMT>(o, s, w[i0 + i][0], w[i0 + i][1]);
            *reinterpret_cast<v2u*>(q + (r0 + i0 + i) * I + tc) = v2u{w[i0 + i][0], w[i0 + i][1]};
        }
    }
    narrow_write_transposed(w, qt + (int64_t)tc * M + r0, M);
}

// One element per lane: small shapes, and ragged ones that are narrow or have few rows (edge_worth, codes_kind_of).
// h, partial, q and qt may be NULL.
template <int QFMT>
__global__ __launch_bounds__(kSwThreads) void swiglu_fwd_elements_kernel(
    const uint16_t* __restrict__ gu, int64_t M, int64_t I, uint16_t* __restrict__ h,
    unsigned* __restrict__ partial, const float* __restrict__ d_qscale, uint8_t* __restrict__ q, uint8_t* __restrict__ qt) {
    __shared__ unsigned s_part[kSwThreads / kWave];
    const int64_t n = M * I;
    unsigned mag = 0;
    float s = 0.0f;
    if constexpr (QFMT >= 0) s = *d_qscale;
    for (int64_t idx = (int64_t)blockIdx.x * kSwThreads + threadIdx.x; idx < n; idx += (int64_t)gridDim.x * kSwThreads) {
        const int64_t m = idx / I, i = idx - m * I;
        const float g = __uint_as_float((unsigned)gu[m * 2 * I + i] << 16);
        const float u = __uint_as_float((unsigned)gu[m * 2 * I + I + i] << 16);
        const unsigned bits = pack_bf16(swiglu_f32<false>(g, u), 0.0f) & 0xFFFFu;
        if (h) h[idx] = (uint16_t)bits;
        mag = pk_max_mag(mag, bits);
        if constexpr (QFMT >= 0) {
            const float p = __uint_as_float(bits << 16) * s;
            const uint8_t code = (uint8_t)(cvt_pair<QFMT>(p, p, 0u, false) & 0xFFu);
            q[idx] = code;
            if (qt) qt[i * M + m] = code;
        }
    }
    if (partial) {
        mag = block_max_u32<kSwThreads>(mag & 0xFFFFu, s_part);
        if (threadIdx.x == 0) partial[blockIdx.x] = mag;
    }
}

__global__ __launch_bounds__(kSwThreads) void swiglu_bwd_elements_kernel(
    const uint16_t* __restrict__ dh, const uint16_t* __restrict__ gu, int64_t M, int64_t I,
    uint16_t* __restrict__ dgu, unsigned* __restrict__ partial) {
    __shared__ unsigned s_part[kSwThreads / kWave];
    const int64_t n = M * I;
    unsigned mag = 0;
    for (int64_t idx = (int64_t)blockIdx.x * kSwThreads + threadIdx.x; idx < n; idx += (int64_t)gridDim.x * kSwThreads) {
        const int64_t m = idx / I, i = idx - m * I;
        const float g = __uint_as_float((unsigned)gu[m * 2 * I + i] << 16);
        const float u = __uint_as_float((unsigned)gu[m * 2 * I + I + i] << 16);
        const float d = __uint_as_float((unsigned)dh[idx] << 16);
        float dg, du;
        swiglu_bwd_f32<false>(d, g, u, dg, du);
        const unsigned w = pack_bf16(dg, du);
        dgu[m * 2 * I + i] = (uint16_t)(w & 0xFFFFu);
        dgu[m * 2 * I + I + i] = (uint16_t)(w >> 16);
        mag = pk_max_mag(mag, w);
    }
    mag = (mag & 0xFFFFu) > (mag >> 16) ? (mag & 0xFFFFu) : (mag >> 16);
    mag = block_max_u32<kSwThreads>(mag, s_part);
    if (threadIdx.x == 0) partial[blockIdx.x] = mag;
}

static bool patch_ok(int64_t M, int64_t I, int pr) { return M % pr == 0 && I % 8 == 0; }

// Ragged shapes: workgroups of an absmax-producing launch, at most one per word of the scratch
static int64_t edge_col_pieces(int64_t I) { return (I + kSwEdgeCols - 1) / kSwEdgeCols; }
static int64_t edge_pieces(int64_t M, int64_t I) { return ((M + kSwEdgeRows - 1) / kSwEdgeRows) * edge_col_pieces(I); }
static int64_t edge_scratch_words(int64_t M, int64_t I) {
    const int64_t b = (M * I + kSwThreads - 1) / kSwThreads;
    return b > kSwEdgeMaxBlocks ? kSwEdgeMaxBlocks : b;
}
static int64_t edge_blocks(int64_t M, int64_t I) {
    const int64_t b = (edge_pieces(M, I) + kSwThreads / kWave - 1) / (kSwThreads / kWave), w = edge_scratch_words(M, I);
    const int64_t trips = (b + w - 1) / w;             // the same number of pieces for every workgroup, give or take one
    return (b + trips - 1) / trips;
}

// Which kernel ragged (and small or narrow) shapes take: one element per lane, or guarded vectors once there is enough to move
// for their code and their waits.  Microseconds, elements / vectors, two to six sets of buffers in turn:
//   forward with h   1001 x 600 6.3 / 7.0, 2001 x 600 7.3 / 7.1, 4001 x 200 6.6 / 7.0, 8001 x 200 8.3 / 7.9, 8001 x 264 8.9 / 8.1,
//                    200001 x 264 156 / 93;  rows that are no whole vectors 1000 x 1001 7.0 / 7.4, 4001 x 500 9.2 / 8.2, 1001 x 2001 9.5 / 8.3, 8000 x 300
//                    10.2 / 9.6, 2001 x 1366 11.3 / 10.1, 4001 x 1001 13.9 / 10.5, 4001 x 2730 37 / 20, 60001 x 100 19 / 35
//   backward         1001 x 2736 11.9 / 11.0, 2001 x 600 7.7 / 8.5, 8001 x 264 11 / 11, 4001 x 200 6.9 / 8.4;  other rows 8000 x 300 10.5 / 12.8, 2001 x 1366
//                    11.7 / 13.3, 4001 x 1001 14.5 / 14.1, 8001 x 515 14.6 / 18.5, 8001 x 701 24.5 / 19.3, 4001 x 2730 42 / 28
//   codes in both layouts   500 x 1000 5.1 / 6.3, 129 x 5001 6.1 / 5.9, 8000 x 100 7.4 / 6.1, 1000 x 1000 8.8 / 7.1, 1000 x 1001 8.7 / 6.3, 250 x 5001 10.3 / 6.9,
//                    4001 x 500 14.7 / 7.3;  33 x 20000 4.8 / 5.9, 60000 x 33 10.3 / 11.7, 16384 x 8 2.2 / 6.0 (narrow patches 13)
//   codes alone      1000 x 1001 4.7 / 6.1, 4001 x 512 6.6 / 5.6, 4001 x 500 6.9 / 6.3, 1001 x 2001 6.9 / 6.4, 8000 x 300 8.1 / 7.6, 4001 x 1001 11.7 / 8.6
// LLMQ_CODES_KERNEL=0 / 1 / 2 (tests): elements, narrow patches or vectors, where they take the shape.
static bool edge_worth(int64_t M, int64_t I, bool backward) {
    if (const char* e = tuning_env("LLMQ_CODES_KERNEL")) return atoi(e) != kCodesElements;
    const int64_t n = M * I;
    if (I % 8 == 0) return I >= (backward ? 256 : 200) && n >= (backward ? (int64_t)3 << 19 : (int64_t)1 << 20);
    // (a wave takes 512 columns.  Elements / vectors, two sets of buffers and twelve: all but full waves, 4 to 5 million elements 1.01 and 1.35, 7 to 8 1.11 and
    // 1.41;  used to 0.6 to 0.7, 5 to 8 million 0.88 and 1.16;  less 0.80 and 1.06, 8 to 11 million 0.92 and 1.23)
    if (backward) {
        const int64_t wave_cols = edge_col_pieces(I) * kSwEdgeCols;
        return I >= 256 && n >= (10 * I >= 7 * wave_cols ? (int64_t)15 << 18 : 100 * I >= 63 * wave_cols ? (int64_t)5 << 20 : (int64_t)1 << 23);
    }
    return I >= 256 && n >= (int64_t)15 << 17;
}
static CodesKind codes_kind_of(int64_t M, int64_t I, bool transpose) {
    if (const char* e = tuning_env("LLMQ_CODES_KERNEL")) {
        const int k = atoi(e);
        return k != kCodesNarrow ? (CodesKind)k : transpose && codes_narrow_ok(M, I) ? kCodesNarrow : kCodesSmall;
    }
    const int64_t n = M * I;
    // (two sets of buffers and twelve, elements / tiles: up to 512 columns, 1.75 to 2 million elements 0.82 and 0.87, 2 to 2.36 0.93 and 0.94, 2.36 to 3 1.10 and
    // 1.03;  more columns 1.75 to 2 0.95 and 0.98, 2 to 2.36 1.03 and 1.01)
    if (!transpose) return M >= 32 && I >= 64 && n >= (I < 512 ? (int64_t)9 << 18 : (int64_t)15 << 17) ? kCodesSmall : kCodesElements;
    if (I >= 32 && n >= ((int64_t)1 << 22) && codes_narrow_ok(M, I)) return kCodesNarrow;       // 1000000 x 32: 105 / 81 / 107 us
    return M >= 32 && I >= 64 && n >= (int64_t)3 << 18 ? kCodesSmall : kCodesElements;
}

// Workgroups of the absmax-producing launches (forward with h, backward): an upper bound of the partial
// results written, which is what the scratch is sized for.
int64_t swiglu_blocks(int64_t M, int64_t I) {
    if (!patch_ok(M, I, 4)) return edge_scratch_words(M, I);
    return ((M + 4 * kSwLanesR - 1) / (4 * kSwLanesR)) * ((I + kSwBlockCols - 1) / kSwBlockCols);
}

static int64_t patch_blocks(int64_t M, int64_t I, int pr) {
    return ((M + pr * kSwLanesR - 1) / (pr * kSwLanesR)) * ((I + kSwBlockCols - 1) / kSwBlockCols);
}

template <int PR, bool WRITE_H, bool AMAX, int QFMT, bool STREAM = false>
static void launch_fwd_patch(const uint16_t* gu, int64_t M, int64_t I, uint16_t* h, unsigned* partial,
                             const float* d_qscale, uint8_t* q, hipStream_t stream) {
    const unsigned gr = (unsigned)((M + PR * kSwLanesR - 1) / (PR * kSwLanesR)), gc = (unsigned)((I + kSwBlockCols - 1) / kSwBlockCols);
    hipLaunchKernelGGL((swiglu_fwd_patch_kernel<PR, WRITE_H, AMAX, QFMT, STREAM>), dim3(gr * gc), dim3(kSwThreads), 0, stream,
                       gu, M, I, h, partial, d_qscale, q, gc);
}

template <int QFMT>
static int launch_fwd_fp8(const uint16_t* gu, int64_t M, int64_t I, uint16_t* h, const float* d_qscale,
                          uint8_t* q, uint8_t* q_t, hipStream_t stream, bool qt_slabs) {
    if (qt_slabs && !(q_t && slab_shape_ok(M, I))) return -2;
    const int64_t row_stride = qt_slabs ? kTileRows : M, band_stride = qt_slabs ? I * kTileRows : kTileRows;
    if (q_t && takes_large_tile(M, I, h ? kSwigluOutputTiles : kSwigluTiles)) {
        const unsigned gr = (unsigned)(M / kTileRows), gc = (unsigned)(I / kTileCols);
        auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3(gr * gc), dim3(kTileThreads), 0, stream, gu, I, h, d_qscale, q, q_t, gc, row_stride, band_stride); };
        if (streams_out(2 * M * I, I, 128)) { if (h) launch(swiglu_fwd_tile_kernel<true, QFMT, true>); else launch(swiglu_fwd_tile_kernel<false, QFMT, true>); }
        else { if (h) launch(swiglu_fwd_tile_kernel<true, QFMT, false>); else launch(swiglu_fwd_tile_kernel<false, QFMT, false>); }
    } else if (!q_t && patch_ok(M, I, 4)) {
        if (h) launch_fwd_patch<4, true, false, QFMT>(gu, M, I, h, nullptr, d_qscale, q, stream);
        else launch_fwd_patch<4, false, false, QFMT>(gu, M, I, h, nullptr, d_qscale, q, stream);
    } else if (const CodesKind kind = qt_slabs ? kCodesSmall : codes_kind_of(M, I, q_t != nullptr); kind == kCodesElements) {
        hipLaunchKernelGGL((swiglu_fwd_elements_kernel<QFMT>), dim3((unsigned)edge_scratch_words(M, I)), dim3(kSwThreads), 0, stream, gu, M, I, h,
                           (unsigned*)nullptr, d_qscale, q, q_t);
    } else if (kind == kCodesNarrow) {
        hipLaunchKernelGGL(swiglu_fwd_fp8_narrow_kernel<QFMT>, dim3((unsigned)((M + kNarrowRows - 1) / kNarrowRows)), dim3(kSwThreads), 0, stream,
                           gu, M, I, h, d_qscale, q, q_t);
    } else {
        small_launches(small_grid(M, I, false, q_t != nullptr), [&](const SmallGrid& g, unsigned blocks) {
            if (q_t) hipLaunchKernelGGL((swiglu_fwd_fp8_small_kernel<QFMT, true>), dim3(blocks), dim3(kTileThreads), 0, stream, gu, M, I, h, d_qscale, q, q_t, g, row_stride, band_stride);
            else hipLaunchKernelGGL((swiglu_fwd_fp8_small_kernel<QFMT, false>), dim3(blocks), dim3(kTileThreads), 0, stream, gu, M, I, h, d_qscale, q, q_t, g, row_stride, band_stride);
        });
    }
    return 0;
}

int launch_swiglu_fwd(const void* gu_, int64_t M, int64_t I, void* h_, unsigned* partial, int amax_fmt,
                      float* d_amax, float* d_scale, const float* d_qscale, int q_fmt, uint8_t* q, uint8_t* q_t,
                      hipStream_t stream, bool qt_slabs) {
    const uint16_t* gu = reinterpret_cast<const uint16_t*>(gu_);
    uint16_t* h = reinterpret_cast<uint16_t*>(h_);
    if (q) {                                   // absmax known: FP8 bytes directly, h optional
        const int st = q_fmt == 0 ? launch_fwd_fp8<0>(gu, M, I, h, d_qscale, q, q_t, stream, qt_slabs)
                                  : launch_fwd_fp8<1>(gu, M, I, h, d_qscale, q, q_t, stream, qt_slabs);
        if (st != 0) return st;
        return hipGetLastError() == hipSuccess ? 0 : -6;
    }
    if (qt_slabs) return -2;
    int64_t n_partial;
    if (patch_ok(M, I, 8)) {                   // 8 rows per lane: more bytes in flight, half the partial results
        if (streams_out(2 * M * I, I, 64)) launch_fwd_patch<8, true, true, -1, true>(gu, M, I, h, partial, nullptr, nullptr, stream);
        else launch_fwd_patch<8, true, true, -1>(gu, M, I, h, partial, nullptr, nullptr, stream);
        n_partial = patch_blocks(M, I, 8);
    } else if (patch_ok(M, I, 4)) {
        launch_fwd_patch<4, true, true, -1>(gu, M, I, h, partial, nullptr, nullptr, stream);
        n_partial = patch_blocks(M, I, 4);
    } else if (!edge_worth(M, I, false)) {
        n_partial = edge_scratch_words(M, I);
        hipLaunchKernelGGL((swiglu_fwd_elements_kernel<-1>), dim3((unsigned)n_partial), dim3(kSwThreads), 0, stream, gu, M, I, h, partial,
                           (const float*)nullptr, (uint8_t*)nullptr, (uint8_t*)nullptr);
    } else {
        n_partial = edge_blocks(M, I);
        hipLaunchKernelGGL(swiglu_fwd_edge_kernel, dim3((unsigned)n_partial), dim3(kSwThreads), 0, stream, gu, M, I, h, partial,
                           (unsigned)edge_col_pieces(I), edge_pieces(M, I));
    }
    if (hipGetLastError() != hipSuccess) return -6;
    return launch_amax_final(partial, (int)n_partial, amax_fmt, d_amax, d_scale, stream);
}

int launch_swiglu_bwd(const void* dh, const void* gu, int64_t M, int64_t I, void* dgu, unsigned* partial,
                      int amax_fmt, float* d_amax, float* d_scale, hipStream_t stream) {
    int64_t n_partial = swiglu_blocks(M, I);
    // (a wave of the patch kernel is 64 columns wide: patches / elements: 16384 x 16 8.0 / 4.6 us, 60000 x 16 9.8 / 6.5, 1000000 x 16 81 / 43)
    const bool narrow = I <= 32 || !patch_ok(M, I, 4);
    if (!narrow) {
        const unsigned gr = (unsigned)((M + 4 * kSwLanesR - 1) / (4 * kSwLanesR)), gc = (unsigned)((I + kSwBlockCols - 1) / kSwBlockCols);
        auto launch = [&](auto kernel) {
            hipLaunchKernelGGL(kernel, dim3(gr * gc), dim3(kSwThreads), 0, stream, reinterpret_cast<const uint16_t*>(dh),
                               reinterpret_cast<const uint16_t*>(gu), M, I, reinterpret_cast<uint16_t*>(dgu), partial, gc);
        };
        if (streams_out(4 * M * I, I, 64)) launch(swiglu_bwd_patch_kernel<true>); else launch(swiglu_bwd_patch_kernel<false>);
    } else if (patch_ok(M, I, 4) || !edge_worth(M, I, true)) {
        if (edge_scratch_words(M, I) < n_partial) n_partial = edge_scratch_words(M, I);
        hipLaunchKernelGGL(swiglu_bwd_elements_kernel, dim3((unsigned)n_partial), dim3(kSwThreads), 0, stream, reinterpret_cast<const uint16_t*>(dh),
                           reinterpret_cast<const uint16_t*>(gu), M, I, reinterpret_cast<uint16_t*>(dgu), partial);
    } else {
        n_partial = edge_blocks(M, I);
        hipLaunchKernelGGL(swiglu_bwd_edge_kernel, dim3((unsigned)n_partial), dim3(kSwThreads), 0, stream,
                           reinterpret_cast<const uint16_t*>(dh), reinterpret_cast<const uint16_t*>(gu), M, I,
                           reinterpret_cast<uint16_t*>(dgu), partial, (unsigned)edge_col_pieces(I),
                           edge_pieces(M, I));
    }
    if (hipGetLastError() != hipSuccess) return -6;
    return launch_amax_final(partial, (int)n_partial, amax_fmt, d_amax, d_scale, stream);
}

}  // namespace llmq
