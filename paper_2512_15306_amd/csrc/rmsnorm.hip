// RMSNorm joined with the residual addition, with the extra outputs of the FP8 pipeline (paper
// Section 3, kernel-fusion paragraph: RMS-norm and residual-stream addition are one kernel that also
// returns the absmax of the normalised output; Section 3 "Activation checkpointing": with the
// statistics kept from the forward pass, the FP8 conversion is fused in during recomputation).
//
//   res'[m,c] = bf16( res[m,c] + x[m,c] ),  rstd[m] = 1 / sqrt( mean_c res'[m,c]^2 + eps ),
//   y[m,c]    = bf16( (res'[m,c] * rstd[m]) * w[c] )
//
// Forward kernels: one wavefront per row, or a workgroup on two rows at a time; the row stays in registers between the
// reduction and the normalisation (one pass over HBM: 4 B read, 2 + 2 B written per element; 2 B less without the
// addition), sum of squares in binary32 with a butterfly over the lanes, absmax of y as a packed
// integer max of the rounded bits, one partial absmax per workgroup for the second-stage kernel.
// The order of that sum is a function of C alone, so that a row has the same statistic whichever kernel and batch it is
// computed in, and so do the codes made from it:
//   C % 8 == 0, C <= 8192:        lane l of 64 adds up the vectors of eight elements l, l + 64, l + 128, ... one after the other;
//   other C <= 2048 or > 16384:   lane l adds up the elements l, l + 64, l + 128, ...;
//   the rest:                     four waves add up the vectors l, l + 256, l + 512, ... of theirs (l = 64 wave + lane), the first
//                                 wave's sum first;
// each wave's 64 sums by a butterfly.  Kernels whose lanes hold other parts of a row pass it through LDS.
// Recompute kernels: rstd and the scale are inputs, so the operation is element-wise; they have the
// lane geometry of the quantize kernels and reuse their transposes to write the FP8 codes in both layouts (2 B read,
// 1 + 1 B written per element).
#include <stdlib.h>

#include "llmq_device.h"
#include "llmq_kernels.h"

#pragma clang fp contract(off)

namespace llmq {
template <int N> struct IntTag { static constexpr int value = N; };

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float v2f __attribute__((ext_vector_type(2)));

constexpr int kRnThreads = 256;
constexpr int kRnRowsPerBlock = kRnThreads / kWave;        // one wavefront per row
constexpr int64_t kRnVecOrderC = 8192;                      // widest row that one wave sums vector by vector

__device__ inline unsigned rn_pack(float lo, float hi) {
    v2f v = {lo, hi};
    return __builtin_bit_cast(unsigned, __builtin_convertvector(v, bf16x2));
}
__device__ inline float rn_lo(unsigned w) { return __uint_as_float(w << 16); }
__device__ inline float rn_hi(unsigned w) { return __uint_as_float(w & 0xFFFF0000u); }

__device__ inline float wave_sum_f32(float v) {
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, kWave);
    return v;
}

__device__ inline void add_squares(const v4u& r, float& ss) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const float a = rn_lo(r[j]), b = rn_hi(r[j]);
        ss = __builtin_fmaf(a, a, ss);
        ss = __builtin_fmaf(b, b, ss);
    }
}
// The same element by element, from a row in LDS
__device__ inline float sum_by_elements(const uint16_t* s_row, int C, int lane) {
    float ss = 0.0f;
#pragma unroll 8
    for (int c = lane; c < C; c += kWave) {
        const float v = __uint_as_float((unsigned)s_row[c] << 16);
        ss = __builtin_fmaf(v, v, ss);
    }
    return ss;
}

__device__ inline unsigned fold_pairs(unsigned m0, unsigned m1, unsigned m2, unsigned m3) {
    m0 = pk_max_mag(pk_max_mag(m0, m1), pk_max_mag(m2, m3));
    return (m0 & 0xFFFFu) > (m0 >> 16) ? (m0 & 0xFFFFu) : (m0 >> 16);
}

// y = bf16((r * rstd) * w) for the eight elements of one 16-byte vector
__device__ inline v4u normalize8(const v4u& r, float rstd, const v4u& w) {
    v4u o;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const float a = rn_lo(r[j]) * rstd, b = rn_hi(r[j]) * rstd;
        o[j] = rn_pack(a * rn_lo(w[j]), b * rn_hi(w[j]));
    }
    return o;
}

// The first `valid` of eight elements, zeros for the others: what lies behind the end of a row counts for nothing, also where
// 0 * rstd * w is NaN (a row whose squares underflow, eps = 0: rstd is infinite and the row's own results are too).
__device__ inline v4u keep_upto(v4u v, int valid) {
#pragma unroll
    for (int j = 0; j < 4; ++j) v[j] &= (2 * j < valid ? 0xFFFFu : 0u) | (2 * j + 1 < valid ? 0xFFFF0000u : 0u);
    return v;
}

// Vector idx of a row of C elements; EDGE: of any C, at any even address
template <bool EDGE>
__device__ inline v4u rn_load(const uint16_t* row, int idx, int C) {
    if constexpr (!EDGE) return __builtin_nontemporal_load(reinterpret_cast<const v4u*>(row) + idx);
    if (8 * idx + 8 <= C) return __builtin_nontemporal_load(reinterpret_cast<const v4u_at2*>(row + 8 * idx));
    return load8_upto(row + 8 * idx, 8 * idx, C - 8 * idx);
}
// Rows of more than 2048 columns: every vector is loaded at once, the last one as the row's last eight elements, and shifted where it is used
// (rn_last), by one branch that the other vectors' lanes skip together.  With the shift beside each load (rn_load) a lane of eight vectors and their
// addition took 279 registers, now 128, and 7616 x 9885 325 us (161 with the last vector loaded element by element, 137 so); 4001 x 10001 169 (83,
// 76), without the addition 70 (42, 41).
__device__ inline const v4u_at2* rn_vector(const uint16_t* row, unsigned at, int C) {       // (32-bit offsets from a uniform address)
    const unsigned end = 2u * (unsigned)(C - 8);
    return reinterpret_cast<const v4u_at2*>(reinterpret_cast<const uint8_t*>(row) + (at < end ? at : end));
}
template <bool EDGE>
__device__ inline v4u rn_load_wide(const uint16_t* row, int idx, unsigned at, int C) {
    if constexpr (!EDGE) return __builtin_nontemporal_load(reinterpret_cast<const v4u*>(row) + idx);
    return __builtin_nontemporal_load(rn_vector(row, at, C));
}
template <bool EDGE, bool STREAM>
__device__ inline void rn_store_wide(uint16_t* row, int idx, unsigned at, int last, int C, const v4u& v) {
    if constexpr (!EDGE) store_hinted<STREAM>(v, reinterpret_cast<v4u*>(row) + idx);
    else if (idx < last) *reinterpret_cast<v4u_at2*>(reinterpret_cast<uint8_t*>(row) + at) = v;
    else store8_upto(row + 8 * last, v, C - 8 * last);
}
// k: vector idx of the row is the lane's k-th
template <bool EDGE>
__device__ inline void rn_last(v4u& v, int k, int last, int C) {
    if constexpr (EDGE) {
        if (k == last / kRnThreads && (int)threadIdx.x == last % kRnThreads) v = shift_elements(v, 8 * last + 8 - C);
    }
}
template <bool EDGE, bool STREAM = false>
__device__ inline void rn_store(uint16_t* row, int idx, int C, const v4u& v) {
    if constexpr (!EDGE) store_hinted<STREAM>(v, reinterpret_cast<v4u*>(row) + idx);
    else store8_upto(row + 8 * idx, v, C - 8 * idx);
}

// One wavefront per row, VPL vectors per lane in registers.  EDGE: any C (the rows start at any even address, the last
// vector of a row may be a part of one); else C % 8 == 0.  HAS_X false: no addition (res is normalised as it is, res_out is not
// written).
template <bool HAS_X, bool EDGE, int VPL>
__global__ __launch_bounds__(kRnThreads) void rmsnorm_row_kernel(
    const uint16_t* res, const uint16_t* __restrict__ x, const uint16_t* __restrict__ w,
    int64_t M, int C, float eps, uint16_t* res_out, uint16_t* __restrict__ y,
    float* __restrict__ rstd_out, unsigned* __restrict__ partial) {
    // res_out may be res (addition in place): every lane reads its elements before it writes them
    __shared__ unsigned s_part[kRnThreads / kWave];
    __shared__ v4u s_rows[kRnRowsPerBlock][EDGE ? VPL * kWave : 1];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x / kWave;
    const int64_t row = (int64_t)blockIdx.x * kRnRowsPerBlock + wave;
    const int nvec = EDGE ? (C + 7) / 8 : C / 8;
    unsigned mag = 0;
    auto load = [&](const uint16_t* base, int idx) { return rn_load<EDGE>(base, idx, C); };
    auto store = [&](uint16_t* base, int idx, const v4u& v) { rn_store<EDGE>(base, idx, C, v); };
    if (row < M) {
        const uint16_t* pr = res + row * C;
        const uint16_t* px = HAS_X ? x + row * C : nullptr;
        v4u r[VPL];
#pragma unroll
        for (int k = 0; k < VPL; ++k) {
            const int idx = k * kWave + lane;
            if (k * kWave < nvec && idx < nvec) {
                r[k] = load(pr, idx);
                if constexpr (HAS_X) {
                    const v4u xv = load(px, idx);
#pragma unroll
                    for (int j = 0; j < 4; ++j)
                        r[k][j] = rn_pack(rn_lo(r[k][j]) + rn_lo(xv[j]), rn_hi(r[k][j]) + rn_hi(xv[j]));
                }
            }
        }
        float ss = 0.0f;
#pragma unroll
        for (int k = 0; k < VPL; ++k) {
            const int idx = k * kWave + lane;
            if (k * kWave < nvec && idx < nvec) {
                if constexpr (HAS_X) store(res_out + row * C, idx, r[k]);
                if constexpr (EDGE) s_rows[wave][idx] = r[k];
                else add_squares(r[k], ss);
            }
        }
        if constexpr (EDGE) {
            // only this wave reads what it wrote: no barrier, but the order of its LDS accesses has to stay
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
            ss = sum_by_elements(reinterpret_cast<const uint16_t*>(s_rows[wave]), C, lane);
        }
        ss = wave_sum_f32(ss);
        const float ms = ss / (float)C;
        const float rstd = 1.0f / __builtin_sqrtf(ms + eps);
        if (lane == 0) rstd_out[row] = rstd;
        unsigned m0 = 0, m1 = 0, m2 = 0, m3 = 0;
#pragma unroll
        for (int k = 0; k < VPL; ++k) {
            const int idx = k * kWave + lane;
            if (k * kWave < nvec && idx < nvec) {
                v4u wv;
                if constexpr (EDGE) wv = load8_upto(w + 8 * idx, 8 * idx, C - 8 * idx);
                else wv = reinterpret_cast<const v4u*>(w)[idx];
                v4u o = normalize8(r[k], rstd, wv);
                if (EDGE && idx == nvec - 1) o = keep_upto(o, C % 8);
                store(y + row * C, idx, o);
                m0 = pk_max_mag(m0, o[0]);
                m1 = pk_max_mag(m1, o[1]);
                m2 = pk_max_mag(m2, o[2]);
                m3 = pk_max_mag(m3, o[3]);
            }
        }
        mag = fold_pairs(m0, m1, m2, m3);
    }
    mag = block_max_u32<kRnThreads>(mag, s_part);
    if (threadIdx.x == 0) partial[blockIdx.x] = mag;
}

// Wider rows: the four rows of a workgroup are read by all of its lanes (VPL vectors per lane and row, two rows at a time),
// so that a lane holds a few vectors of each row instead of a whole row's share, which leaves room for more waves, and
// reads the norm's weight once for both.  Where one wave adds up the squares of a row, it reads them from LDS; widths that had
// no kernel of one wave per row to agree with are summed by all four (by one, element by element, 4001 x 10001 took 102 us
// instead of 73).  Measured against
// one wave per row with up to 16 vectors per lane, with the addition: 16384 x 5120 137 -> 130 us (5.2 TB/s), 8192 x 3584
// 52 -> 46, 4096 x 7680 59 -> 51, 279 x 7680 21 -> 14; all four rows at a time took 134, 48, 63 and 14.
template <bool HAS_X, bool EDGE, int VPL, bool STREAM>
__global__ __launch_bounds__(kRnThreads) void rmsnorm_rows_kernel(
    const uint16_t* res, const uint16_t* __restrict__ x, const uint16_t* __restrict__ w,
    int64_t M, int C, float eps, uint16_t* res_out, uint16_t* __restrict__ y,
    float* __restrict__ rstd_out, unsigned* __restrict__ partial) {
    constexpr int ROWS = VPL <= 4 ? 2 : 1;
    constexpr bool ONE_WAVE = !EDGE && VPL * kRnThreads * 8 <= kRnVecOrderC;        // sums a row (VPL > 4 is for wider ones)
    constexpr int kWaves = kRnThreads / kWave;
    __shared__ unsigned s_part[kWaves];
    __shared__ float s_rstd[kRnRowsPerBlock], s_sum[kRnRowsPerBlock][kWaves];
    __shared__ v4u s_rows[ONE_WAVE ? ROWS : 1][ONE_WAVE ? VPL * kRnThreads : 1];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x / kWave;
    const int nvec = EDGE ? (C + 7) / 8 : C / 8;
    unsigned m0 = 0, m1 = 0, m2 = 0, m3 = 0;
#pragma unroll 1
    for (int p = 0; p < kRnRowsPerBlock; p += ROWS) {
        const int64_t row = (int64_t)blockIdx.x * kRnRowsPerBlock + p;
        if (row >= M) break;                                 // the same for the whole workgroup
        // Byte offset of the lane's k-th vector.  Opaque in every trip, or the compiler keeps an address for each vector of each tensor across them.
        unsigned lane_at = 16u * threadIdx.x;
        if constexpr (EDGE) asm volatile("" : "+v"(lane_at));
        auto at = [&](int k) { return lane_at + (unsigned)(k * kRnThreads * 16); };
        v4u r[ROWS][VPL], xv[ROWS][HAS_X ? VPL : 1];
#pragma unroll
        for (int i = 0; i < ROWS; ++i)
#pragma unroll
            for (int k = 0; k < VPL; ++k) {
                const int idx = k * kRnThreads + threadIdx.x;
                r[i][k] = v4u{0, 0, 0, 0};
                if (row + i < M && idx < nvec) {
                    r[i][k] = rn_load_wide<EDGE>(res + (row + i) * C, idx, at(k), C);
                    if constexpr (HAS_X) xv[i][k] = rn_load_wide<EDGE>(x + (row + i) * C, idx, at(k), C);
                }
            }
#pragma unroll
        for (int i = 0; i < ROWS; ++i) {
            float ss = 0.0f;
#pragma unroll
            for (int k = 0; k < VPL; ++k) {
                const int idx = k * kRnThreads + threadIdx.x;
                if (row + i < M && idx < nvec) {
                    rn_last<EDGE>(r[i][k], k, nvec - 1, C);
                    if constexpr (HAS_X) {
                        rn_last<EDGE>(xv[i][k], k, nvec - 1, C);
#pragma unroll
                        for (int j = 0; j < 4; ++j)
                            r[i][k][j] = rn_pack(rn_lo(r[i][k][j]) + rn_lo(xv[i][k][j]), rn_hi(r[i][k][j]) + rn_hi(xv[i][k][j]));
                        rn_store_wide<EDGE, STREAM>(res_out + (row + i) * C, idx, at(k), nvec - 1, C, r[i][k]);
                    }
                    if constexpr (ONE_WAVE) s_rows[i][idx] = r[i][k];
                    else add_squares(r[i][k], ss);
                }
            }
            if constexpr (!ONE_WAVE) {
                ss = wave_sum_f32(ss);
                if (lane == 0) s_sum[p + i][wave] = ss;
            }
        }
        __syncthreads();
        float rstd[ROWS];
        if constexpr (ONE_WAVE) {
            if (wave < ROWS && row + wave < M) {
                float ss = 0.0f;
#pragma unroll 4
                for (int idx = lane; idx < nvec; idx += kWave) add_squares(s_rows[wave][idx], ss);
                ss = wave_sum_f32(ss);
                const float ms = ss / (float)C;
                const float t = 1.0f / __builtin_sqrtf(ms + eps);
                if (lane == 0) {
                    rstd_out[row + wave] = t;
                    s_rstd[p + wave] = t;
                }
            }
            __syncthreads();
#pragma unroll
            for (int i = 0; i < ROWS; ++i) rstd[i] = s_rstd[p + i];
        } else {
#pragma unroll
            for (int i = 0; i < ROWS; ++i) {
                float t = s_sum[p + i][0];
#pragma unroll
                for (int v = 1; v < kWaves; ++v) t += s_sum[p + i][v];
                const float ms = t / (float)C;
                rstd[i] = 1.0f / __builtin_sqrtf(ms + eps);
                if (threadIdx.x == 0 && row + i < M) rstd_out[row + i] = rstd[i];
            }
        }
#pragma unroll
        for (int k = 0; k < VPL; ++k) {
            const int idx = k * kRnThreads + threadIdx.x;
            if (idx < nvec) {
                v4u wv;
                if constexpr (EDGE) wv = *rn_vector(w, at(k), C);
                else wv = reinterpret_cast<const v4u*>(w)[idx];
                rn_last<EDGE>(wv, k, nvec - 1, C);
#pragma unroll
                for (int i = 0; i < ROWS; ++i)
                    if (row + i < M) {
                        v4u o = normalize8(r[i][k], rstd[i], wv);
                        if (EDGE && idx == nvec - 1) o = keep_upto(o, C % 8);
                        rn_store_wide<EDGE, STREAM>(y + (row + i) * C, idx, at(k), nvec - 1, C, o);
                        m0 = pk_max_mag(m0, o[0]);
                        m1 = pk_max_mag(m1, o[1]);
                        m2 = pk_max_mag(m2, o[2]);
                        m3 = pk_max_mag(m3, o[3]);
                    }
            }
        }
    }
    const unsigned mag = block_max_u32<kRnThreads>(fold_pairs(m0, m1, m2, m3), s_part);
    if (threadIdx.x == 0) partial[blockIdx.x] = mag;
}

// More than 16384 columns: one wavefront per row, element-wise strided loops; the row is read again for the second pass
// (from res_out when the addition was done).
__global__ __launch_bounds__(kRnThreads) void rmsnorm_row_generic_kernel(
    const uint16_t* res, const uint16_t* __restrict__ x, const uint16_t* __restrict__ w,
    int64_t M, int64_t C, float eps, uint16_t* res_out, uint16_t* __restrict__ y,
    float* __restrict__ rstd_out, unsigned* __restrict__ partial) {
    __shared__ unsigned s_part[kRnThreads / kWave];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x / kWave;
    const int64_t row = (int64_t)blockIdx.x * kRnRowsPerBlock + wave;
    unsigned mag = 0;
    if (row < M) {
        float ss = 0.0f;
        for (int64_t c = lane; c < C; c += kWave) {
            unsigned bits = res[row * C + c];
            if (x) {
                bits = rn_pack(__uint_as_float(bits << 16) + __uint_as_float((unsigned)x[row * C + c] << 16), 0.0f) & 0xFFFFu;
                res_out[row * C + c] = (uint16_t)bits;
            }
            const float v = __uint_as_float(bits << 16);
            ss = __builtin_fmaf(v, v, ss);
        }
        ss = wave_sum_f32(ss);
        const float ms = ss / (float)C;
        const float rstd = 1.0f / __builtin_sqrtf(ms + eps);
        if (lane == 0) rstd_out[row] = rstd;
        const uint16_t* src = x ? res_out : res;          // this lane re-reads exactly the elements it wrote
        for (int64_t c = lane; c < C; c += kWave) {
            const float t = __uint_as_float((unsigned)src[row * C + c] << 16) * rstd;
            const unsigned o = rn_pack(t * __uint_as_float((unsigned)w[c] << 16), 0.0f) & 0xFFFFu;
            y[row * C + c] = (uint16_t)o;
            mag = pk_max_mag(mag, o);
        }
    }
    mag = block_max_u32<kRnThreads>(mag & 0xFFFFu, s_part);
    if (threadIdx.x == 0) partial[blockIdx.x] = mag;
}

// Recompute path: rstd [M] and the scale are given, no transposed copy.  Lane = 4 rows x 8 columns; M % 4 == 0, C % 8 == 0.
constexpr int kRnLanesR = 8;
constexpr int kRnBlockCols = 8 * (kWave / kRnLanesR) * (kRnThreads / kWave);

template <int QFMT, bool WRITE_Y>
__global__ __launch_bounds__(kRnThreads) void rmsnorm_apply_fp8_patch_kernel(
    const uint16_t* __restrict__ res, const uint16_t* __restrict__ w, const float* __restrict__ rstd,
    int64_t M, int64_t C, const float* __restrict__ d_qscale, uint8_t* __restrict__ q, uint16_t* __restrict__ y,
    unsigned grid_cols) {
    constexpr int PR = 4;
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x / kWave;
    const unsigned brow = blockIdx.x / grid_cols, bcol = blockIdx.x % grid_cols;     // walk along the columns
    const int64_t r0 = (int64_t)brow * (PR * kRnLanesR) + (lane % kRnLanesR) * PR;
    const int64_t c0 = (int64_t)bcol * kRnBlockCols + wave * (8 * (kWave / kRnLanesR)) + (lane / kRnLanesR) * 8;
    if (r0 >= M || c0 >= C) return;
    const uint16_t* src = res + r0 * C + c0;
    v4u in[PR];
#pragma unroll
    for (int i = 0; i < PR; ++i) in[i] = __builtin_nontemporal_load(reinterpret_cast<const v4u*>(src + (int64_t)i * C));
    const v4u wv = *reinterpret_cast<const v4u*>(w + c0);
    const v4f rs = *reinterpret_cast<const v4f*>(rstd + r0);
    const float s = *d_qscale;
    uint8_t* dq = q + r0 * C + c0;
#pragma unroll
    for (int i = 0; i < PR; ++i) {
        const v4u o = normalize8(in[i], rs[i], wv);
        if constexpr (WRITE_Y) *reinterpret_cast<v4u*>(y + (r0 + i) * C + c0) = o;
        unsigned lo, hi;
        quantize8<QFMT>(o, s, lo, hi);
        *reinterpret_cast<v2u*>(dq + (int64_t)i * C) = v2u{lo, hi};
    }
}

// With the transposed copy, tensors made of whole 128 x 128 tiles: lane geometry and LDS transpose of the quantize kernel's tile
// variant (full 128-byte lines on every stream; the transposed copy optionally in slabs).
template <int QFMT, bool WRITE_Y, bool STREAM>
__global__ __launch_bounds__(kTileThreads) void rmsnorm_apply_fp8_tile_kernel(
    const uint16_t* __restrict__ res, const uint16_t* __restrict__ w, const float* __restrict__ rstd,
    int64_t C, const float* __restrict__ d_qscale, uint8_t* __restrict__ q,
    uint8_t* __restrict__ qt, uint16_t* __restrict__ y, unsigned grid_cols, int64_t qt_row_stride,
    int64_t qt_band_stride) {
    __shared__ __attribute__((aligned(16))) uint8_t s_t[kTileLdsBytes];
    const unsigned brow = blockIdx.x / grid_cols, bcol = blockIdx.x - brow * grid_cols;   // along the columns first
    int tr, tc;
    tile_patch_origin(tr, tc);
    const int64_t r0 = (int64_t)brow * kTileRows + tr, c0 = (int64_t)bcol * kTileCols + tc;
    const uint16_t* src = res + r0 * C + c0;
    v4u in[kPatchRows];
#pragma unroll
    for (int i = 0; i < kPatchRows; ++i) in[i] = __builtin_nontemporal_load(reinterpret_cast<const v4u*>(src + (int64_t)i * C));
    const v4u wv = *reinterpret_cast<const v4u*>(w + c0);
    float rs[kPatchRows];
#pragma unroll
    for (int i = 0; i < kPatchRows / 4; ++i) {
        const v4f t = *reinterpret_cast<const v4f*>(rstd + r0 + 4 * i);
        rs[4 * i] = t[0]; rs[4 * i + 1] = t[1]; rs[4 * i + 2] = t[2]; rs[4 * i + 3] = t[3];
    }
    const float s = *d_qscale;
    __builtin_amdgcn_sched_barrier(0);
    unsigned wq[kPatchRows][2];
#pragma unroll
    for (int i = 0; i < kPatchRows; ++i) {
        const v4u o = normalize8(in[i], rs[i], wv);
        if constexpr (WRITE_Y) *reinterpret_cast<v4u*>(y + (r0 + i) * C + c0) = o;
        quantize8<QFMT>(o, s, wq[i][0], wq[i][1]);
    }
    uint8_t* dq = q + r0 * C + c0;
#pragma unroll
    for (int i = 0; i < kPatchRows; ++i) store_hinted<STREAM>(v2u{wq[i][0], wq[i][1]}, reinterpret_cast<v2u*>(dq + (int64_t)i * C));
    tile_stage_transposed(wq, tr, tc, s_t);
    __syncthreads();
    tile_write_transposed(s_t, qt + (int64_t)bcol * kTileCols * qt_row_stride + (int64_t)brow * qt_band_stride, qt_row_stride);
}

// Narrow shapes of whole 16 x 8 patches, with the transposed copy (codes_kind; 64 x 128 tile / patches: 60000 x 64 7.7 / 6.1 us,
// 1000000 x 16 49 / 28).  y may be NULL.
template <int QFMT>
__global__ __launch_bounds__(kRnThreads) void rmsnorm_apply_fp8_narrow_kernel(
    const uint16_t* __restrict__ res, const uint16_t* __restrict__ w, const float* __restrict__ rstd,
    int64_t M, int64_t C, const float* __restrict__ d_qscale, uint8_t* __restrict__ q,
    uint8_t* __restrict__ qt, uint16_t* __restrict__ y) {
    int tr, tc;
    narrow_patch_origin(tr, tc);
    const int64_t r0 = (int64_t)blockIdx.x * kNarrowRows + tr;
    if (r0 >= M || tc >= C) return;
    const uint16_t* src = res + r0 * C + tc;
    v4u in[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) in[i] = __builtin_nontemporal_load(reinterpret_cast<const v4u*>(src + (int64_t)i * C));
    const v4u wv = *reinterpret_cast<const v4u*>(w + tc);
    v4f rs[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) rs[i] = *reinterpret_cast<const v4f*>(rstd + r0 + 4 * i);
    const float s = *d_qscale;
    unsigned wq[16][2];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const v4u o = normalize8(in[i], rs[i / 4][i % 4], wv);
        if (y) *reinterpret_cast<v4u*>(y + (r0 + i) * C + tc) = o;
        quantize8<QFMT>(o, s, wq[i][0], wq[i][1]);
    }
    uint8_t* dq = q + r0 * C + tc;
#pragma unroll
    for (int i = 0; i < 16; ++i) *reinterpret_cast<v2u*>(dq + (int64_t)i * C) = v2u{wq[i][0], wq[i][1]};
    narrow_write_transposed(wq, qt + (int64_t)tc * M + r0, M);
}

// One element per lane: small shapes, and ragged ones that are narrow or have few rows.  qt, y may be NULL.
constexpr int64_t kApplyElementsMaxBlocks = 65536;
template <int QFMT>
__global__ __launch_bounds__(kRnThreads) void rmsnorm_apply_fp8_elements_kernel(
    const uint16_t* __restrict__ res, const uint16_t* __restrict__ w, const float* __restrict__ rstd,
    int64_t M, int64_t C, const float* __restrict__ d_qscale, uint8_t* __restrict__ q,
    uint8_t* __restrict__ qt, uint16_t* __restrict__ y) {
    const int64_t n = M * C;
    const float s = *d_qscale;
    for (int64_t idx = (int64_t)blockIdx.x * kRnThreads + threadIdx.x; idx < n; idx += (int64_t)gridDim.x * kRnThreads) {
        const int64_t m = idx / C, c = idx - m * C;
        const float t = __uint_as_float((unsigned)res[idx] << 16) * rstd[m];
        const unsigned bits = rn_pack(t * __uint_as_float((unsigned)w[c] << 16), 0.0f) & 0xFFFFu;
        if (y) y[idx] = (uint16_t)bits;
        const float p = __uint_as_float(bits << 16) * s;
        const uint8_t code = (uint8_t)(cvt_pair<QFMT>(p, p, 0u, false) & 0xFFu);
        q[idx] = code;
        if (qt) qt[c * M + m] = code;
    }
}

// Ragged shapes and tensors of few tiles: the 64 x 128 tile; y (if not NULL), q and the transposed copy (TRANSPOSE).
template <int QFMT, bool TRANSPOSE>
__global__ __launch_bounds__(kTileThreads) void rmsnorm_apply_fp8_small_kernel(
    const uint16_t* __restrict__ res, const uint16_t* __restrict__ w, const float* __restrict__ rstd,
    int64_t M, int64_t C, const float* __restrict__ d_qscale, uint8_t* __restrict__ q,
    uint8_t* __restrict__ qt, uint16_t* __restrict__ y, const SmallGrid grid, int64_t qt_row_stride, int64_t qt_band_stride) {
    __shared__ __attribute__((aligned(16))) uint8_t s_t[TRANSPOSE ? kSmallLdsBytes : 16];
    unsigned brow, bcol;
    if (!small_tile(grid, grid.first + blockIdx.x, brow, bcol)) return;
    int tr, tc;
    small_patch_origin(grid, tr, tc);
    const int64_t R0 = (int64_t)brow * kSmallRows, C0 = (int64_t)bcol * kSmallCols, r0 = R0 + tr, c0 = C0 + tc;
    with_guard(small_tile_guard(R0, C0, M, C), [&](auto guard) {
        const int64_t rows_left = guard ? M - r0 : kSmallPatch, cols_left = guard ? C - c0 : 8;
        v4u in[kSmallPatch];
        v4u wv[1];
        load_tile_patches_upto(c0, rows_left, cols_left, patch(in, res + r0 * C + c0, C), shared_row(wv, w + c0));
        float rs[kSmallPatch];
#pragma unroll
        for (int i = 0; i < kSmallPatch; ++i) rs[i] = i < rows_left ? rstd[r0 + i] : 0.0f;
        const float s = *d_qscale;
        unsigned wq[kSmallPatch][2];
#pragma unroll
        for (int i = 0; i < kSmallPatch; ++i) {
            in[i] = normalize8(in[i], rs[i], wv[0]);
            quantize8<QFMT>(in[i], s, wq[i][0], wq[i][1]);
        }
        if (y) store_patch_upto(in, y + r0 * C + c0, C, rows_left, cols_left);
        store_codes_upto(wq, q + r0 * C + c0, C, rows_left, cols_left);
        if constexpr (TRANSPOSE) {
            small_stage_transposed(wq, tr, tc, s_t);
            __syncthreads();
            small_write_transposed_upto(s_t, qt + C0 * qt_row_stride + (R0 / kTileRows) * qt_band_stride + R0 % kTileRows, qt_row_stride,
                                        guard ? M - R0 : kSmallRows, guard ? C - C0 : kSmallCols);
        }
    });
}

int64_t rmsnorm_blocks(int64_t M) { return (M + kRnRowsPerBlock - 1) / kRnRowsPerBlock; }

// Which forward kernel.  Microseconds with the addition unless said otherwise (generic: element by element, a wave per row;
// row: vectors, a wave per row; rows: the workgroup reads its rows together).
//   Rows of whole vectors up to 2048 columns, generic against row: 4001 x 264 8.8 / 6.6, 16384 x 1000 33 / 29: always row.
//   Ragged rows, generic against row: 16384 x 100 10.5 / 14.7, 2048 x 300 7.7 / 7.7, 4001 x 385 10.1 / 8.9, 16384 x 1001 42 / 32;
//   without the addition and on many rows the generic kernel, which has less to move then, holds out longer: 16384 x 501 17 / 21,
//   60001 x 700 65 / 79, 8001 x 701 11.9 / 13.7, 16384 x 1001 30 / 26, while 4001 x 450 takes 8.7 / 8.3.
//   Wide rows, row against rows; "cold" with buffers of its own for every pass, "warm" with the same ones:
//     cold 126 x 2304 9.8 / 9.2, 126 x 3072 11.1 / 9.6, 126 x 3584 12.3 / 9.9, 126 x 7168 18.4 / 14.4, 640 x 5120 17.0 / 13.8,
//     1536 x 8192 30.5 / 27.2, 2048 x 4096 18.9 / 18.8, 3000 x 5120 27.6 / 30.5, 4096 x 3584 25.7 / 28.6, 8000 x 7168 95.6 / 90.6,
//     16384 x 4096 110 / 94; warm 126 x 2304 7.0 / 8.4, 126 x 3072 7.5 / 8.8, 126 x 3584 8.1 / 9.1, 126 x 7168 11.6 / 12.9,
//     640 x 5120 11.4 / 12.0, 1536 x 8192 31.5 / 26.3, 3000 x 5120 27.3 / 28.3, 16384 x 5120 134 / 124.  The line is where rows gains
//     at least twice as much cold as it loses warm, or gains in both.  One or two rows are faster with rows at any width, 1 x 8192 9.9 / 6.2.
//     Without the addition a wave has half as much to wait for, and row is faster from three rows on: cold 126 x 7168 8.8 / 10.6,
//     3000 x 5120 15.0 / 18.4, 16384 x 7168 90.9 / 86.9, warm 81.8 / 86.0.
//   More than 8192 columns, or ragged and more than 2048: rows at any size (300 x 8200 55 / 18 against generic).
// LLMQ_NORM_KERNEL=0 / 1 / 2 (tests): generic, row or rows wherever that kernel takes the width.
enum NormKind { kNormGeneric, kNormRow, kNormRows };
static NormKind norm_kind(int64_t M, int64_t C, bool with_x) {
    const bool edge = C % 8 != 0;
    const bool row_ok = C <= 4 * kWave * 8 || (!edge && C <= 16 * kWave * 8), rows_ok = C > 4 * kWave * 8 && C <= 8 * kRnThreads * 8;
    const bool generic_ok = edge ? C <= 4 * kWave * 8 : !rows_ok && !row_ok;       // by the order of the sums
    if (const char* e = tuning_env("LLMQ_NORM_KERNEL")) {
        const int k = atoi(e);
        if (k == 0 && generic_ok) return kNormGeneric;
        if (k == 1 && row_ok) return kNormRow;
        if (k == 2 && rows_ok) return kNormRows;
    }
    if (!row_ok) return rows_ok ? kNormRows : kNormGeneric;
    if (edge) return C < (with_x ? 320 : M >= 6000 ? 800 : 384) ? kNormGeneric : kNormRow;
    if (!rows_ok) return kNormRow;
    return M <= 2 || (with_x && C > 3072 && (M < 2560 || M >= 12288)) ? kNormRows : kNormRow;
}

int launch_rmsnorm_fwd(const void* res_, const void* x_, const void* w_, int64_t M, int64_t C, float eps,
                       void* res_out_, void* y_, float* rstd, unsigned* partial, int fmt, float* d_amax,
                       float* d_scale, hipStream_t stream) {
    const uint16_t* res = reinterpret_cast<const uint16_t*>(res_);
    const uint16_t* x = reinterpret_cast<const uint16_t*>(x_);
    const uint16_t* w = reinterpret_cast<const uint16_t*>(w_);
    uint16_t* res_out = reinterpret_cast<uint16_t*>(res_out_);
    uint16_t* y = reinterpret_cast<uint16_t*>(y_);
    const dim3 grid((unsigned)rmsnorm_blocks(M)), block(kRnThreads);
    auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, block, 0, stream, res, x, w, M, (int)C, eps, res_out, y, rstd, partial); };
    const bool edge = C % 8 != 0;
    auto row = [&](auto vpl) {
        constexpr int V = decltype(vpl)::value;
        if constexpr (V <= 4) {                            // (ragged rows of more vectors per lane take the rows kernel)
            if (edge) { if (x) launch(rmsnorm_row_kernel<true, true, V>); else launch(rmsnorm_row_kernel<false, true, V>); return; }
        }
        if (x) launch(rmsnorm_row_kernel<true, false, V>); else launch(rmsnorm_row_kernel<false, false, V>);
    };
    auto rows = [&](auto vpl) {
        constexpr int V = decltype(vpl)::value;
        const bool out = streams_out((x ? 4 : 2) * M * C, C, 64);
        if (x) { if (edge) launch(rmsnorm_rows_kernel<true, true, V, false>); else if (out) launch(rmsnorm_rows_kernel<true, false, V, true>); else launch(rmsnorm_rows_kernel<true, false, V, false>); }
        else { if (edge) launch(rmsnorm_rows_kernel<false, true, V, false>); else if (out) launch(rmsnorm_rows_kernel<false, false, V, true>); else launch(rmsnorm_rows_kernel<false, false, V, false>); }
    };
    switch (norm_kind(M, C, x != nullptr)) {
        case kNormGeneric: hipLaunchKernelGGL(rmsnorm_row_generic_kernel, grid, block, 0, stream, res, x, w, M, C, eps, res_out, y, rstd, partial); break;
        case kNormRow:
            // (As few registers as the row needs, but for a few workgroups per CU: those are dealt out evenly only if few fit
            // on one.  3000 x 3584 with 8 and 16 vectors per lane: 21.4 / 19.1 us, 4001 x 3584 24.7 / 29.4.)
            if (C <= 4 * kWave * 8) row(IntTag<4>{});
            else if (x && M >= 1280 && M <= 3500) row(IntTag<16>{});
            else if (C <= 8 * kWave * 8) row(IntTag<8>{});
            else if (C <= 12 * kWave * 8) row(IntTag<12>{});
            else row(IntTag<16>{});
            break;
        case kNormRows:
            if (C <= 2 * kRnThreads * 8) rows(IntTag<2>{});
            else if (C <= 3 * kRnThreads * 8) rows(IntTag<3>{});
            else if (C <= 4 * kRnThreads * 8) rows(IntTag<4>{});
            else rows(IntTag<8>{});
    }
    if (hipGetLastError() != hipSuccess) return -6;
    return launch_amax_final(partial, (int)rmsnorm_blocks(M), fmt, d_amax, d_scale, stream);
}

// The recompute call's kernel where it is not the large tile's or, without the transposed copy, that of whole 4 x 8 patches.
// Without the transposed copy the 64 x 128 tile is worth its code and its waits only for millions of elements (elements / tile,
// microseconds: 250 x 5001 3.7 / 3.9, 4001 x 500 4.9 / 4.2, 1001 x 2001 4.9 / 4.3, 2001 x 1366 7.0 / 5.1, 4001 x 512 5.1 / 4.1, 4001 x 2730 21 / 10, 4001 x 200 3.8 / 4.7,
// 200001 x 33 11.3 / 14.4).
static CodesKind apply_kind(int64_t M, int64_t C, bool transpose) {
    if (transpose) return codes_kind(M, C);
    if (const char* e = tuning_env("LLMQ_CODES_KERNEL")) return atoi(e) == 0 ? kCodesElements : kCodesSmall;
    return M >= 32 && C >= 64 && M * C >= (int64_t)15 << 17 ? kCodesSmall : kCodesElements;
}

template <int QFMT>
static void launch_apply(const uint16_t* res, const uint16_t* w, const float* rstd, int64_t M, int64_t C,
                         const float* d_qscale, uint8_t* q, uint8_t* q_t, uint16_t* y, hipStream_t stream,
                         bool qt_slabs) {
    const int64_t row_stride = qt_slabs ? kTileRows : M, band_stride = qt_slabs ? C * kTileRows : kTileRows;
    if (q_t && takes_large_tile(M, C, y ? kNormOutputTiles : kNormTiles)) {
        const unsigned tr = (unsigned)(M / kTileRows), tcn = (unsigned)(C / kTileCols);
        auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3(tr * tcn), dim3(kTileThreads), 0, stream, res, w, rstd, C, d_qscale, q, q_t, y, tcn, row_stride, band_stride); };
        if (streams_out(2 * M * C, C, 128)) { if (y) launch(rmsnorm_apply_fp8_tile_kernel<QFMT, true, true>); else launch(rmsnorm_apply_fp8_tile_kernel<QFMT, false, true>); }
        else { if (y) launch(rmsnorm_apply_fp8_tile_kernel<QFMT, true, false>); else launch(rmsnorm_apply_fp8_tile_kernel<QFMT, false, false>); }
    } else if (!q_t && M % 4 == 0 && C % 8 == 0) {
        const unsigned gc = (unsigned)((C + kRnBlockCols - 1) / kRnBlockCols);
        const dim3 grid((unsigned)((M + 4 * kRnLanesR - 1) / (4 * kRnLanesR)) * gc);
        if (y) hipLaunchKernelGGL((rmsnorm_apply_fp8_patch_kernel<QFMT, true>), grid, dim3(kRnThreads), 0, stream, res, w, rstd, M, C, d_qscale, q, y, gc);
        else hipLaunchKernelGGL((rmsnorm_apply_fp8_patch_kernel<QFMT, false>), grid, dim3(kRnThreads), 0, stream, res, w, rstd, M, C, d_qscale, q, y, gc);
    } else if (const CodesKind kind = qt_slabs ? kCodesSmall : apply_kind(M, C, q_t != nullptr); kind == kCodesElements) {
        const int64_t blocks = (M * C + kRnThreads - 1) / kRnThreads;
        const dim3 grid((unsigned)(blocks < kApplyElementsMaxBlocks ? blocks : kApplyElementsMaxBlocks));
        hipLaunchKernelGGL(rmsnorm_apply_fp8_elements_kernel<QFMT>, grid, dim3(kRnThreads), 0, stream, res, w, rstd, M, C, d_qscale, q, q_t, y);
    } else if (kind == kCodesNarrow) {
        hipLaunchKernelGGL(rmsnorm_apply_fp8_narrow_kernel<QFMT>, dim3((unsigned)((M + kNarrowRows - 1) / kNarrowRows)), dim3(kRnThreads), 0, stream,
                           res, w, rstd, M, C, d_qscale, q, q_t, y);
    } else {
        small_launches(small_grid(M, C, false, q_t != nullptr), [&](const SmallGrid& g, unsigned blocks) {
            if (q_t) hipLaunchKernelGGL((rmsnorm_apply_fp8_small_kernel<QFMT, true>), dim3(blocks), dim3(kTileThreads), 0, stream, res, w, rstd, M, C, d_qscale, q, q_t, y, g, row_stride, band_stride);
            else hipLaunchKernelGGL((rmsnorm_apply_fp8_small_kernel<QFMT, false>), dim3(blocks), dim3(kTileThreads), 0, stream, res, w, rstd, M, C, d_qscale, q, q_t, y, g, row_stride, band_stride);
        });
    }
}

int launch_rmsnorm_apply_fp8(const void* res, const void* w, const float* rstd, int64_t M, int64_t C,
                             const float* d_qscale, int fmt, uint8_t* q, uint8_t* q_t, void* y, hipStream_t stream,
                             bool qt_slabs) {
    const uint16_t* r = reinterpret_cast<const uint16_t*>(res);
    const uint16_t* wp = reinterpret_cast<const uint16_t*>(w);
    if (qt_slabs && !(q_t && slab_shape_ok(M, C))) return -2;
    if (fmt == 0) launch_apply<0>(r, wp, rstd, M, C, d_qscale, q, q_t, reinterpret_cast<uint16_t*>(y), stream, qt_slabs);
    else launch_apply<1>(r, wp, rstd, M, C, d_qscale, q, q_t, reinterpret_cast<uint16_t*>(y), stream, qt_slabs);
    return hipGetLastError() == hipSuccess ? 0 : -6;
}

}  // namespace llmq
