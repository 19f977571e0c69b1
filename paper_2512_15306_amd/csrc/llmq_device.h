// Device-side helpers shared by the gfx950 kernels of the FP8 linear path.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <type_traits>

#include "llmq_kernels.h"

namespace llmq {

typedef int v2i __attribute__((ext_vector_type(2)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef int v8i __attribute__((ext_vector_type(8)));
typedef unsigned v2u __attribute__((ext_vector_type(2)));
typedef unsigned v4u __attribute__((ext_vector_type(4)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef unsigned short v2us __attribute__((ext_vector_type(2)));

constexpr int kWave = 64;

__host__ __device__ inline float fp8_max(int fmt) { return fmt == 0 ? 448.0f : 57344.0f; }

// Maximum over the 64 lanes of a wavefront: butterfly inside each row of 16 lanes with DPP
// (quad permutes, then the two row mirrors), then the four row results are combined.
__device__ inline unsigned wave_max_u32(unsigned v) {
    unsigned t;
    t = (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xF, 0xF, false);   // quad_perm [1,0,3,2]
    v = v > t ? v : t;
    t = (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xF, 0xF, false);   // quad_perm [2,3,0,1]
    v = v > t ? v : t;
    t = (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xF, 0xF, false);  // row_half_mirror
    v = v > t ? v : t;
    t = (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xF, 0xF, false);  // row_mirror
    v = v > t ? v : t;
    unsigned a = (unsigned)__builtin_amdgcn_readlane((int)v, 0);
    unsigned b = (unsigned)__builtin_amdgcn_readlane((int)v, 16);
    unsigned c = (unsigned)__builtin_amdgcn_readlane((int)v, 32);
    unsigned d = (unsigned)__builtin_amdgcn_readlane((int)v, 48);
    a = a > b ? a : b;
    c = c > d ? c : d;
    return a > c ? a : c;
}

// Magnitude bits of a BF16 absmax -> binary32 bit pattern, NaNs made canonical.
// Non-negative floats order like their bit patterns, so the integer max of these is the float max,
// with NaN (0x7FC00000) above +Inf (0x7F800000) above every finite value.
__device__ inline unsigned amax_bits_from_bf16_mag(unsigned mag16) {
    return mag16 > 0x7F80u ? 0x7FC00000u : (mag16 << 16);
}

// Packed maximum of the magnitudes (bits & 0x7FFF) of the two BF16 values in w with the pair in acc.
__device__ inline unsigned pk_max_mag(unsigned acc, unsigned w) {
    v2us a = __builtin_bit_cast(v2us, acc);
    v2us b = __builtin_bit_cast(v2us, w & 0x7FFF7FFFu);
    return __builtin_bit_cast(unsigned, __builtin_elementwise_max(a, b));
}

__device__ inline unsigned pk_max_u16(unsigned a, unsigned b) {
    return __builtin_bit_cast(unsigned, __builtin_elementwise_max(__builtin_bit_cast(v2us, a), __builtin_bit_cast(v2us, b)));
}

// Maximum over a workgroup of THREADS lanes; s_part holds one word per wavefront.
template <int THREADS>
__device__ inline unsigned block_max_u32(unsigned m, unsigned* s_part) {
    m = wave_max_u32(m);
    if ((threadIdx.x & (kWave - 1)) == 0) s_part[threadIdx.x / kWave] = m;
    __syncthreads();
#pragma unroll
    for (int w = 0; w < THREADS / kWave; ++w) m = m > s_part[w] ? m : s_part[w];
    return m;
}

// The scale of a tensor whose absmax is a (paper Section 3 "Overview": the absmax is mapped onto the largest
// finite FP8 value): fmax / a with one correctly rounded binary32 division, FLT_MAX when that quotient
// overflows (a tiny absmax), and 1 for an all-zero tensor, where the rule defines nothing and every scale
// gives the same codes (+-0): the neutral scale keeps the de-scaling exact and stays usable as a kept statistic.
// a = +Inf gives 0, a = NaN gives NaN.
__device__ inline float scale_of_amax(float a, float fmax) {
    float s = fmax / a;
    if (__builtin_isinf(s)) s = a == 0.0f ? 1.0f : 3.402823466e+38f;
    return s;
}

// The same from a BF16 magnitude pattern, as the absmax second stage computes it
__device__ inline float scale_from_mag(unsigned mag16, float fmax) {
    return scale_of_amax(__uint_as_float(amax_bits_from_bf16_mag(mag16)), fmax);
}

// The scale of a 256-lane workgroup's launch; all lanes of the workgroup must call it.
__device__ inline float resolve_scale(const ScaleSource& src, bool first_block, unsigned* s_part) {
    if (src.partial == nullptr) return *src.d_scale;
    unsigned m = 0;
    for (int i = threadIdx.x; i < src.n_partial; i += 256) {
        const unsigned v = src.partial[i];
        m = m > v ? m : v;
    }
    m = block_max_u32<256>(m, s_part);
    const float s = scale_from_mag(m, src.fmax);
    if (first_block && threadIdx.x == 0) *src.d_scale_out = s;
    return s;
}

// Workgroup id -> block (brow, bcol) of a grid of grid_rows x grid_cols blocks: bands of `band` block columns
// (1 <= band <= grid_cols, so that band * grid_rows stays within the grid size, which fits 32 bits), walked down
// the rows, `band` neighbouring blocks of a row one after the other; the last band takes the columns that are
// left.  band = 1: down the rows; band = grid_cols: along the columns.
__host__ __device__ inline void band_walk(unsigned id, unsigned grid_rows, unsigned grid_cols, unsigned band,
                                          unsigned& brow, unsigned& bcol) {
    const unsigned band_first = (id / (band * grid_rows)) * band;
    const unsigned band_width = grid_cols - band_first < band ? grid_cols - band_first : band;
    const unsigned in_band = id - band_first * grid_rows;
    brow = in_band / band_width;
    bcol = band_first + in_band % band_width;
}

// A store, with the streaming hint if STREAM
template <bool STREAM, class T>
__device__ inline void store_hinted(const T& v, T* p) {
    if constexpr (STREAM) __builtin_nontemporal_store(v, p);
    else *p = v;
}

// ---- FP8 cast helpers (used by the quantize kernel and by the producers that emit FP8 directly) ----

template <int FMT>
__device__ inline unsigned cvt_pair(float a, float b, unsigned old, bool high) {
    constexpr float fmax = FMT == 0 ? 448.0f : 57344.0f;
    a = __builtin_amdgcn_fmed3f(a, -fmax, fmax);         // saturate; the cast below rounds to nearest even
    b = __builtin_amdgcn_fmed3f(b, -fmax, fmax);
    if constexpr (FMT == 0) {
        return high ? (unsigned)__builtin_amdgcn_cvt_pk_fp8_f32(a, b, (int)old, true)
                    : (unsigned)__builtin_amdgcn_cvt_pk_fp8_f32(a, b, (int)old, false);
    } else {
        return high ? (unsigned)__builtin_amdgcn_cvt_pk_bf8_f32(a, b, (int)old, true)
                    : (unsigned)__builtin_amdgcn_cvt_pk_bf8_f32(a, b, (int)old, false);
    }
}

// Four BF16 pairs (one 16-byte load) -> eight FP8 codes in two dwords.
template <int FMT>
__device__ inline void quantize8(const v4u& r, float s, unsigned& lo, unsigned& hi) {
    float f[8];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        f[2 * j] = __uint_as_float(r[j] << 16) * s;            // even element: low half of the dword
        f[2 * j + 1] = __uint_as_float(r[j] & 0xFFFF0000u) * s;
    }
    lo = cvt_pair<FMT>(f[0], f[1], 0u, false);
    lo = cvt_pair<FMT>(f[2], f[3], lo, true);
    hi = cvt_pair<FMT>(f[4], f[5], 0u, false);
    hi = cvt_pair<FMT>(f[6], f[7], hi, true);
}

// w[r] holds bytes (r,0..3) of a 4x4 byte block; returns o[c] = bytes (0..3,c).
__device__ inline void transpose4x4_bytes(const unsigned w[4], unsigned o[4]) {
    // v_perm_b32 selects from the 8 bytes {first operand: 4..7, second operand: 0..3}
    unsigned t01l = __builtin_amdgcn_perm(w[1], w[0], 0x05010400u);   // w0.0 w1.0 w0.1 w1.1
    unsigned t01h = __builtin_amdgcn_perm(w[1], w[0], 0x07030602u);   // w0.2 w1.2 w0.3 w1.3
    unsigned t23l = __builtin_amdgcn_perm(w[3], w[2], 0x05010400u);
    unsigned t23h = __builtin_amdgcn_perm(w[3], w[2], 0x07030602u);
    o[0] = __builtin_amdgcn_perm(t23l, t01l, 0x05040100u);
    o[1] = __builtin_amdgcn_perm(t23l, t01l, 0x07060302u);
    o[2] = __builtin_amdgcn_perm(t23h, t01h, 0x05040100u);
    o[3] = __builtin_amdgcn_perm(t23h, t01h, 0x07060302u);
}

// ---- The 16 x 8 patch without LDS, of the kernels that write FP8 codes of narrow tensors in both layouts ----
//
// Eight lanes stacked (128 rows, whole lines of the transposed tensor) x eight side by side (64 columns), the waves of a
// workgroup side by side: most of them leave at once, which costs less than 512 rows per workgroup on a quarter as many CUs
// (quantize kernel, 60000 x 64: 5.4 / 6.9 us).  rows % 16 == 0 and cols % 8 == 0: a patch is all inside or all outside.
constexpr int kNarrowRows = 128;
__device__ inline void narrow_patch_origin(int& tr, int& tc) {
    const int lane = threadIdx.x & (kWave - 1);
    tr = (lane & 7) * 16;
    tc = (threadIdx.x / kWave) * 64 + (lane >> 3) * 8;
}
// The patch as FP8 bytes, w[row][k] = columns 4k .. 4k+3, to the transposed tensor: column j becomes 16 bytes at dt + j ld.
__device__ inline void narrow_write_transposed(const unsigned (&w)[16][2], uint8_t* dt, int64_t ld) {
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        unsigned col[4][4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const unsigned blk[4] = {w[4 * t][k], w[4 * t + 1][k], w[4 * t + 2][k], w[4 * t + 3][k]};
            unsigned o[4];
            transpose4x4_bytes(blk, o);
#pragma unroll
            for (int c = 0; c < 4; ++c) col[c][t] = o[c];
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) *reinterpret_cast<v4u*>(dt + (int64_t)(4 * k + c) * ld) = v4u{col[c][0], col[c][1], col[c][2], col[c][3]};
    }
}

// ---- The 128 x 128 workgroup tile of the kernels that write FP8 codes in both layouts ----
//
// 256 lanes; a lane owns a patch of 8 rows x 8 columns, a wave is 4 lanes stacked x 16 side by side (32 rows x 128
// columns: its loads of BF16 input cover 256 contiguous bytes of a row, its stores of codes a whole 128-byte line), the four
// waves are stacked.  Four lanes that follow each other lie side by side: a wave's 8-byte stores of codes are put together from
// neighbouring lanes, and with lanes that follow each other stacked instead every piece of 8 bytes went out by itself
// (quantize kernel, slabs, 8192 x 3584: stacked 25.4 us, two side by side 22.6, four 21.6, eight 22.4, sixteen 21.9; 16-byte loads and stores do not
// care).  The transposed patches (8-byte column pieces after the register transpose) go through a
// [128 columns][128 rows] byte tile in LDS (rows padded to 136 bytes against bank conflicts) and
// leave, after one barrier, as 128-byte lines of the transposed tensor, 8 lanes per transposed row.
// With 16 rows per lane (256 x 128) and with 4 (64 x 128) with the same lanes the same tensor took 23.2 and 24.6 us, 3584 x 18944
// 52.8 and 56.0 against 50.1: fewer rows leave shorter lines of the transposed copy, more rows fewer waves per CU.
constexpr int kTileCols = 128, kPatchRows = 8;
constexpr int kTilePitch = kTileRows + 8;         // kTileRows = 128
constexpr int kTileThreads = 256;
constexpr int kTileLdsBytes = kTileCols * kTilePitch;

// Row and column group of a lane in a wave of 4 x 16 patches
__device__ inline void wave_patch(int& stacked, int& beside) {
    const int lane = threadIdx.x & (kWave - 1);
    stacked = (lane >> 2) & 3;
    beside = (lane & 3) | (lane >> 4) << 2;
}

// Origin of this lane's patch inside the tile
__device__ inline void tile_patch_origin(int& tr, int& tc) {
    int stacked, beside;
    wave_patch(stacked, beside);
    tr = (threadIdx.x / kWave) * (4 * kPatchRows) + stacked * kPatchRows;
    tc = beside * 8;
}

// The patch as FP8 bytes, w[row][k] = columns 4k .. 4k+3: column j of the patch becomes 8 consecutive bytes of
// row (tc + j) of the LDS tile, at byte tr.
__device__ inline void tile_stage_transposed(const unsigned (&w)[kPatchRows][2], int tr, int tc, uint8_t* s_t) {
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        unsigned col[4][2];
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            unsigned blk[4] = {w[4 * t][k], w[4 * t + 1][k], w[4 * t + 2][k], w[4 * t + 3][k]};
            unsigned o[4];
            transpose4x4_bytes(blk, o);
#pragma unroll
            for (int c = 0; c < 4; ++c) col[c][t] = o[c];
        }
#pragma unroll
        for (int c = 0; c < 4; ++c)
            *reinterpret_cast<v2u*>(s_t + (tc + 4 * k + c) * kTilePitch + tr) = v2u{col[c][0], col[c][1]};
    }
}

// After the barrier that follows the staging: the whole tile to memory.  dt = where transposed row 0 of this tile
// starts; transposed row c starts row_stride bytes after row c - 1.  The transposed tensor [cols, rows] as such:
// dt = qt + (first column) rows + (first row), row_stride = rows.  In slabs of 128 contraction bytes
// (OperandLayout): dt = qt + (first row / 128) cols 128 + (first column) 128, row_stride = 128, and the tile's
// 16 KB are one contiguous piece.
__device__ inline void tile_write_transposed(const uint8_t* s_t, uint8_t* dt, int64_t row_stride) {
#pragma unroll
    for (int m = 0; m < kTileCols * (kTileRows / 16) / kTileThreads; ++m) {
        const int p = threadIdx.x + m * kTileThreads;       // 16-byte piece: column p / 8, rows 16 (p % 8) ..
        const int c = p >> 3, ch = p & 7;
        const v2u lo = *reinterpret_cast<const v2u*>(s_t + c * kTilePitch + ch * 16), hi = *reinterpret_cast<const v2u*>(s_t + c * kTilePitch + ch * 16 + 8);
        *reinterpret_cast<v4u*>(dt + (int64_t)c * row_stride + ch * 16) = v4u{lo[0], lo[1], hi[0], hi[1]};
    }
}

// ---- The same at the edges of ragged tensors: any number of rows and columns, rows starting at any address ----
//
// A patch that lies inside the tensor moves in the same 16- and 8-byte vectors, only without the alignment (the
// hardware takes them at any address).  Of a vector over the end of a row, the load takes the row's last eight elements instead
// and shifts what belongs to the vector to the front, zeros behind it: loaded element by element, with a wait behind each, the last
// columns' workgroups were what the launch waited for (quantize kernel 4096 x 2730 15.7 us, 4096 x 2728 11.8; now 12.1 and 12.0).
// Only rows of fewer than eight elements are.  The stores move what exists in pieces of four, two and one.
typedef v4u v4u_at2 __attribute__((aligned(2)));
typedef v2u v2u_at2 __attribute__((aligned(2)));
typedef unsigned u32_at2 __attribute__((aligned(2)));
typedef v4u v4u_at1 __attribute__((aligned(1)));
typedef v2u v2u_at1 __attribute__((aligned(1)));
typedef unsigned u32_at1 __attribute__((aligned(1)));
typedef uint16_t u16_at1 __attribute__((aligned(1)));

// The vector moved `drop` elements (0 .. 7) to the front, zeros behind it
__device__ inline v4u shift_elements(const v4u& v, int drop) {
    const int bits = 16 * drop;
    uint64_t lo = ((uint64_t)v[1] << 32) | v[0], hi = ((uint64_t)v[3] << 32) | v[2];
    if (bits >= 64) { lo = hi >> (bits - 64); hi = 0; }
    else if (bits > 0) { lo = (lo >> bits) | (hi << (64 - bits)); hi >>= bits; }
    return v4u{(unsigned)lo, (unsigned)(lo >> 32), (unsigned)hi, (unsigned)(hi >> 32)};
}
__device__ inline v4u load8_by_elements(const uint16_t* p, int64_t valid) {
    v4u v = {0, 0, 0, 0};
#pragma unroll
    for (int e = 0; e < 7; ++e)
        if (e < valid) v[e >> 1] |= (unsigned)p[e] << (16 * (e & 1));
    return v;
}
// Eight BF16 values of a row, from column c0 (a multiple of 8) on, of which the first `valid` exist.
__device__ inline v4u load8_upto(const uint16_t* p, int64_t c0, int64_t valid) {
    if (valid >= 8) return *reinterpret_cast<const v4u_at2*>(p);
    if (valid <= 0) return v4u{0, 0, 0, 0};
    if (c0 < 8) return load8_by_elements(p, valid);
    const int drop = 8 - (int)valid;
    const v4u v = *reinterpret_cast<const v4u_at2*>(p - drop);
    return shift_elements(v, drop);
}
__device__ inline void store8_upto(uint16_t* p, const v4u& v, int64_t valid) {
    if (valid >= 8) { *reinterpret_cast<v4u_at2*>(p) = v; return; }
    if (valid <= 0) return;
    const int n = (int)valid;
    if (n & 4) *reinterpret_cast<v2u_at2*>(p) = v2u{v[0], v[1]};
    const unsigned a = n & 4 ? v[2] : v[0], b = n & 4 ? v[3] : v[1];
    if (n & 2) *reinterpret_cast<u32_at2*>(p + (n & 4)) = a;
    if (n & 1) p[n & 6] = (uint16_t)(n & 2 ? b : a);
}
__device__ inline void store8_codes_upto(uint8_t* p, unsigned lo, unsigned hi, int64_t valid) {
    if (valid >= 8) { *reinterpret_cast<v2u_at1*>(p) = v2u{lo, hi}; return; }
    if (valid <= 0) return;
    const int n = (int)valid;
    if (n & 4) *reinterpret_cast<u32_at1*>(p) = lo;
    const unsigned a = n & 4 ? hi : lo;
    if (n & 2) *reinterpret_cast<u16_at1*>(p + (n & 4)) = (uint16_t)a;
    if (n & 1) p[n & 6] = (uint8_t)(n & 2 ? a >> 16 : a);
}

// The first n (1 .. 15) of sixteen codes
__device__ inline void store16_codes_upto(uint8_t* p, const v4u& v, int n) {
    if (n & 8) *reinterpret_cast<v2u_at1*>(p) = v2u{v[0], v[1]};
    const unsigned lo = n & 8 ? v[2] : v[0], hi = n & 8 ? v[3] : v[1];
    if (n & 7) store8_codes_upto(p + (n & 8), lo, hi, n & 7);
}

// Runs body with a compile-time answer to whether edges have to be guarded.  `guard` is the same for every lane of a wave (of a workgroup, if
// body holds a barrier), so tiles inside the tensor run straight-line code that requests everything before it waits; with the guards'
// branches in the way the patches, the weights and the row factors were waited for one after the other.  Codes, guards per lane / so: SwiGLU
// 8100 x 7168 64.1 / 60.8 us, 12001 x 5000 80.8 / 78.0; RMSNorm 16101 x 4096 52.0 / 46.6, 12001 x 5000 56.6 / 52.1.  One patch and nothing else
// (quantize) has nothing to gain: 8112 x 5128 44.3 / 45.3, 1777 x 2730 6.9 / 7.4; it asks lane by lane.
template <class F>
__device__ inline void with_guard(bool guard, F body) {
    if (guard) body(std::true_type{});
    else body(std::false_type{});
}

// A patch of PR rows x 8 columns of BF16 values at src = column c0 (a multiple of 8) of its first row, rows `ld` elements apart,
// of which rows_left rows and cols_left columns exist.  Patches of several tensors that are guarded alike are requested together: the guards'
// branches, one patch after the other, would wait for each patch before the next one is requested (SwiGLU backward, 9001 x 6001: 155 us
// patch by patch, 131 so; forward 85 / 73).
// SHARED: one row, which the tiles above and below read too, so its loads leave it in the caches (RMSNorm codes behind the forward pass that writes
// their input, the weight read past the caches / so: 4133 x 5120 61.4 / 58.2 us for both calls, 3001 x 5128 47.2 / 44.7, 8263 x 7168 155.8 / 151.7).
template <int PR, bool SHARED>
struct Patch {
    static constexpr int rows = PR;
    v4u (&in)[PR];
    const uint16_t* src;
    int64_t ld;
};
template <int PR>
__device__ inline Patch<PR, false> patch(v4u (&in)[PR], const uint16_t* src, int64_t ld) { return Patch<PR, false>{in, src, ld}; }
__device__ inline Patch<1, true> shared_row(v4u (&in)[1], const uint16_t* src) { return Patch<1, true>{in, src, 0}; }
template <int PR, bool SHARED>
__device__ inline void request_patch(const Patch<PR, SHARED>& p, int drop, int64_t rows_left) {
#pragma unroll
    for (int i = 0; i < PR; ++i) {
        const v4u_at2* src = reinterpret_cast<const v4u_at2*>(p.src - drop + (int64_t)(i < rows_left ? i : 0) * p.ld);
        if constexpr (SHARED) p.in[i] = *src;
        else p.in[i] = __builtin_nontemporal_load(src);
    }
}
template <int PR, bool SHARED>
__device__ inline void shift_patch(const Patch<PR, SHARED>& p, int drop, int64_t rows_left) {
#pragma unroll
    for (int i = 0; i < PR; ++i) p.in[i] = i < rows_left ? shift_elements(p.in[i], drop) : v4u{0, 0, 0, 0};
}
template <int PR, bool SHARED>
__device__ inline void load_patch_by_elements(const Patch<PR, SHARED>& p, int64_t rows_left, int64_t cols_left) {
#pragma unroll
    for (int i = 0; i < PR; ++i) p.in[i] = load8_by_elements(p.src + (int64_t)i * p.ld, i < rows_left ? cols_left : 0);
}
template <int PR, bool SHARED>
__device__ inline void zero_patch(const Patch<PR, SHARED>& p) {
#pragma unroll
    for (int i = 0; i < PR; ++i) p.in[i] = v4u{0, 0, 0, 0};
}
// (of patches of which a row and a column exist)
template <class... P>
__device__ inline void load_patches_upto(int64_t c0, int64_t rows_left, int64_t cols_left, const P&... p) {
    if (cols_left >= 8 || c0 >= 8) {
        const int drop = cols_left >= 8 ? 0 : 8 - (int)cols_left;
        (request_patch(p, drop, rows_left), ...);
        if (((rows_left < P::rows) || ...) || drop != 0) (shift_patch(p, drop, rows_left), ...);
    } else {
        (load_patch_by_elements(p, rows_left, cols_left), ...);
    }
}
// The same of a tile's lanes, whose patches may lie beside the tensor.  Those are zeros at once: as loads of no element of any row, one guard
// after the other, they were what a small launch waited for (patch by patch / requested together / so: RMSNorm codes 1652 x 1024 4.29 / 4.57 / 3.82 us,
// 2275 x 256 4.14 / 4.48 / 3.72; SwiGLU codes 161 x 8192 6.04 / 6.26 / 5.14, 1447 x 856 6.69 / 6.34 / 5.31).
template <class... P>
__device__ inline void load_tile_patches_upto(int64_t c0, int64_t rows_left, int64_t cols_left, const P&... p) {
    if (rows_left > 0 && cols_left > 0) load_patches_upto(c0, rows_left, cols_left, p...);
    else (zero_patch(p), ...);
}
// One patch, where the tile's guard is not known to the whole wave
template <int PR>
__device__ inline void load_patch_upto(v4u (&in)[PR], const uint16_t* src, int64_t ld, int64_t c0, int64_t rows_left, int64_t cols_left) {
    if (rows_left >= PR && cols_left >= 8) {
#pragma unroll
        for (int i = 0; i < PR; ++i) in[i] = __builtin_nontemporal_load(reinterpret_cast<const v4u_at2*>(src + (int64_t)i * ld));
    } else if (rows_left <= 0 || cols_left <= 0) {
#pragma unroll
        for (int i = 0; i < PR; ++i) in[i] = v4u{0, 0, 0, 0};
    } else {
        load_patches_upto(c0, rows_left, cols_left, patch(in, src, ld));
    }
}
template <int PR>
__device__ inline void store_patch_upto(const v4u (&out)[PR], uint16_t* dst, int64_t ld, int64_t rows_left, int64_t cols_left) {
    if (rows_left >= PR && cols_left >= 8) {
#pragma unroll
        for (int i = 0; i < PR; ++i) *reinterpret_cast<v4u_at2*>(dst + (int64_t)i * ld) = out[i];
    } else {
#pragma unroll
        for (int i = 0; i < PR; ++i)
            if (i < rows_left) store8_upto(dst + (int64_t)i * ld, out[i], cols_left);
    }
}
template <int PR>
__device__ inline void store_codes_upto(const unsigned (&w)[PR][2], uint8_t* dst, int64_t ld, int64_t rows_left, int64_t cols_left) {
    if (rows_left >= PR && cols_left >= 8) {
#pragma unroll
        for (int i = 0; i < PR; ++i) *reinterpret_cast<v2u_at1*>(dst + (int64_t)i * ld) = v2u{w[i][0], w[i][1]};
    } else {
#pragma unroll
        for (int i = 0; i < PR; ++i)
            if (i < rows_left) store8_codes_upto(dst + (int64_t)i * ld, w[i][0], w[i][1], cols_left);
    }
}

// ---- The 64-row x 128-column tile of the same kernels for tensors of few tiles ----
//
// A tensor of a few dozen 128 x 128 tiles leaves most of the chip idle.  Here a lane owns 4 rows x 8 columns and twice as many
// workgroups share the tensor; the lanes of a wave lie as above (256-byte runs of the input, whole lines of
// codes; 1024 x 1024 quantized 3.3 us with lanes that follow each other stacked, 3.1 so), the four waves are stacked.  Guarded edges, any
// alignment; the transposed copy leaves in 64-byte pieces.
// (Eight rows per lane with the same guards, 128 x 128: ragged tensors gain nothing or a few percent, 8100 x 5120 38.3 / 37.9 us, 8112 x 5128
// 45.0 / 45.7, 4001 x 2730 16.0 / 18.9, 16000 x 9000 176 / 170.)
constexpr int kSmallRows = 64, kSmallCols = 128, kSmallPatch = 4;
constexpr int kSmallPitch = kSmallRows + 16, kSmallLdsBytes = kSmallCols * kSmallPitch;

// Tiles that share cache lines belong on one XCD (own L2; the hardware deals workgroup ids round-robin to them).  Rows that do not
// start at a line share lines with the tiles beside them, and the lines of the transposed copy, written in 64-byte pieces, are shared with
// the tiles above and below.  In launch order along the columns those above and below lie on the same XCD if a row has a multiple of
// eight tiles, which then is the better order; otherwise each XCD walks a contiguous range of tiles, eight tile columns wide and down the
// rows.  Quantize kernel, launch order / XCD ranges in bands of 2 / 8 / all columns: 8112 x 5128 elements 45.7 / 39.9 / 37.7 / 37.5 us,
// 1777 x 20000 40.3 / 33.5 / 33.6 / 38.9, 9001 x 3001 32.4 / 31.3 / 30.8 / 31.3, 16000 x 9000 202 / 202 / 174 / 173;  launch order / bands of 8, rows of
// whole lines: 56 tiles (8100 x 7168) 53 / 57, 40 (8100 x 5120) 39 / 40, 112 (3333 x 14336) 42 / 42;  220 (6096 x 28160) 232 / 166, 158 (1104 x 20224)
// 25.8 / 22.3, 297 (300 x 38016) 14.1 / 11.9, 22 (4001 x 2816) 14.5 / 12.1, 110 (6096 x 14080) 83 / 82; of less than eight tiles a row either may win.
constexpr unsigned kSmallXcds = 8, kSmallBand = 8;
struct SmallGrid {
    unsigned rows, cols, blocks;            // tiles (at most 2^28: tensors have at most 2^40 elements and 2^31 rows), workgroups in all
    unsigned first;                         // first workgroup of this launch
    bool xcd_ranges;
    bool stacked;                           // lanes that follow each other one above the other instead of side by side
};
// quantizes: for the quantize kernel (and not those that compute what they write as codes); transposed: with the transposed copy.
// Codes alone share lines only where the rows do not start at them, and stacked lanes only make their stores narrower.  RMSNorm codes, three sets of
// buffers in turn, side by side in launch order / in XCD ranges / stacked so: 357 x 16064 5.6 / 5.5 / 6.3 us, 2571 x 8448 14.2 / 13.6 / 15.8,
// 6762 x 2752 12.6 / 12.4 / 14.7, 10134 x 3840 21.0 / 21.6 / 24.2, 12005 x 7488 44.7 / 46.6 / 50.6, 13543 x 9984 71.3 / 83.2 / 86.6;  rows beside the lines 9254 x 7448 49.9 / 42.5 / 44.0,
// 10043 x 14456 156 / 114 / 114.
inline SmallGrid small_grid(int64_t rows, int64_t cols, bool quantizes, bool transposed) {
    SmallGrid g;
    g.rows = (unsigned)((rows + kSmallRows - 1) / kSmallRows);
    g.cols = (unsigned)((cols + kSmallCols - 1) / kSmallCols);
    g.blocks = (g.rows * g.cols + kSmallXcds - 1) / kSmallXcds * kSmallXcds;
    g.first = 0;
    g.xcd_ranges = cols % 64 != 0 || ((transposed || rows * cols <= 20000000) && g.cols > kSmallXcds && g.cols % kSmallXcds != 0);
    // Lanes side by side / stacked, quantize and RMSNorm codes: 1024 x 1024 3.1 / 3.3 and 3.4 / 3.8 us, 4133 x 5120 20.1 / 22.3 and 20.5 /
    // 22.7, two sets of buffers in turn 8100 x 7168 41.3 / 48.6 and 42.7 / 50.0.  Once tensor and codes (4 bytes an element) crowd the 256 MB memory-side
    // cache, stacked lanes take less.  Absmax and quantize of four tensors in turn:
    //   whole vectors, rows that do not start at lines   9001 x 4008 48.6 / 49.8, 11001 x 3912 65.4 / 63.5, 12001 x 5000 102.4 / 95.3, 16221 x 4296 116.8 /
    //     107.9, 16000 x 9000 225.8 / 217.0;  rows of whole lines   8101 x 4416 44.1 / 48.9, 16101 x 4096 85.3 / 84.9, 16101 x 6144 126.9 / 124.1,
    //     9579 x 11200 149.4 / 140.6;  odd widths   6001 x 6001 51.4 / 58.0, 16001 x 8001 189.5 / 194.8, 12001 x 16001 313.9 / 311.2
    // RMSNorm codes, millions of elements 40 to 50 0.92, 60 to 65 0.98, more 1.00 to 1.03, but of odd widths 0.98 to 0.99 throughout;  SwiGLU codes, 6
    // bytes an element, 50 to 60 0.98, more 0.99 to 1.01.
    g.stacked = transposed && cols % 8 == 0 && rows * cols > (int64_t)(quantizes && cols % 64 != 0 ? 40000000 : 66000000);
    return g;
}
// launch(grid, workgroups of this launch), once or as often as the launch limit asks for
template <class F>
inline void small_launches(SmallGrid g, F launch) {
    const unsigned most = max_workgroups();
    for (; g.first < g.blocks; g.first += most) launch(g, g.blocks - g.first < most ? g.blocks - g.first : most);
}
// The tile of workgroup id; false for the padding ids (id 0 always has one)
__host__ __device__ inline bool small_tile(const SmallGrid& g, unsigned id, unsigned& brow, unsigned& bcol) {
    const unsigned pos = g.xcd_ranges ? (id % kSmallXcds) * (g.blocks / kSmallXcds) + id / kSmallXcds : id;
    if (pos >= g.rows * g.cols) return false;
    const unsigned band = g.xcd_ranges && kSmallBand < g.cols ? kSmallBand : g.cols;
    band_walk(pos, g.rows, g.cols, band, brow, bcol);
    return true;
}

// Whether the tile reaches over the tensor's edge
__device__ inline bool small_tile_guard(int64_t R0, int64_t C0, int64_t rows, int64_t cols) {
    return rows - R0 < kSmallRows || cols - C0 < kSmallCols;
}

__device__ inline void small_patch_origin(const SmallGrid& g, int& tr, int& tc) {
    int stacked, beside;
    wave_patch(stacked, beside);
    if (g.stacked) { const int lane = threadIdx.x & (kWave - 1); stacked = lane & 3; beside = lane >> 2; }
    tr = (threadIdx.x / kWave) * 16 + stacked * kSmallPatch;
    tc = beside * 8;
}

__device__ inline void small_stage_transposed(const unsigned (&w)[kSmallPatch][2], int tr, int tc, uint8_t* s_t) {
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const unsigned blk[4] = {w[0][k], w[1][k], w[2][k], w[3][k]};
        unsigned o[4];
        transpose4x4_bytes(blk, o);
#pragma unroll
        for (int c = 0; c < 4; ++c) *reinterpret_cast<unsigned*>(s_t + (tc + 4 * k + c) * kSmallPitch + tr) = o[c];
    }
}

// dt = where row 0 of the tile starts in transposed row 0 of the tile; transposed rows row_stride bytes apart
__device__ inline void small_write_transposed_upto(const uint8_t* s_t, uint8_t* dt, int64_t row_stride, int64_t rows_left, int64_t cols_left) {
#pragma unroll
    for (int m = 0; m < kSmallCols * (kSmallRows / 16) / kTileThreads; ++m) {
        const int p = threadIdx.x + m * kTileThreads;
        const int c = p >> 2, ch = p & 3;
        if (c >= cols_left) continue;
        uint8_t* dst = dt + (int64_t)c * row_stride + ch * 16;
        const int64_t valid = rows_left - ch * 16;
        if (valid <= 0) continue;
        if (valid >= 16) {
            *reinterpret_cast<v4u_at1*>(dst) = *reinterpret_cast<const v4u*>(s_t + c * kSmallPitch + ch * 16);
        } else {
            store16_codes_upto(dst, *reinterpret_cast<const v4u*>(s_t + c * kSmallPitch + ch * 16), (int)valid);
        }
    }
}

}  // namespace llmq
