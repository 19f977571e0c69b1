// Fused scale + FP8 cast + transposed copy (paper Section 3, kernel-fusion paragraph: quantization and
// transposition are one kernel; the FP8 GEMM wants both operands contraction-contiguous, so every
// quantized tensor is also needed transposed in the backward pass).
//
// HBM-bound: per element 2 bytes read, 1 byte written row-major and 1 byte written transposed.  A lane owns a patch of
// 16 rows x 8 columns (4 x 8 in tensors of few tiles): 16-byte loads, one binary32 multiply and the hardware RNE cast
// (clamped first, which makes it saturating), 8-byte stores of each row, a byte transpose in registers with byte
// permutes; the transposed patches leave through LDS in whole pieces of lines.
#include <stdlib.h>

#include "llmq_device.h"
#include "llmq_kernels.h"

namespace llmq {

constexpr int kQThreads = 256;

// Tensors whose rows are a multiple of 128 and whose columns a multiple of 256 (every benchmark tensor): full 128-byte
// lines on all three streams.  A lane owns a 16 x 8 patch, a wave is
// 4 lanes stacked x 16 side by side, and the transposed copy cannot be written that way from registers (4 stacked
// lanes hold 64 contiguous bytes of a transposed row), so the transposed patches go through LDS (the tile_*
// helpers).
template <int FMT, bool STREAM>
__global__ __launch_bounds__(kTileThreads) void quantize_tile_kernel(
    const uint16_t* __restrict__ x, int64_t cols, const ScaleSource scale_src,
    uint8_t* __restrict__ q, uint8_t* __restrict__ qt, unsigned* __restrict__ zero_word, unsigned grid_cols,
    int64_t qt_row_stride, int64_t qt_band_stride) {
    __shared__ unsigned s_part[kTileThreads / kWave];
    __shared__ __attribute__((aligned(16))) uint8_t s_t[kTileLdsBytes];
    if (zero_word && blockIdx.x == 0 && threadIdx.x == 0) *zero_word = 0u;
    // (the scale first: the conversions then follow the loads as they arrive; after them it costs 5 %)
    const float s = resolve_scale(scale_src, blockIdx.x == 0, s_part);
    const unsigned brow = blockIdx.x / grid_cols, bcol = blockIdx.x - brow * grid_cols;   // along the columns first
    int tr, tc;
    tile_patch_origin(tr, tc);
    const int64_t r0 = (int64_t)brow * kTileRows + tr, c0 = (int64_t)bcol * kTileCols + tc;
    v4u in[kPatchRows];
    const uint16_t* src = x + r0 * cols + c0;
#pragma unroll
    for (int i = 0; i < kPatchRows; ++i) in[i] = __builtin_nontemporal_load(reinterpret_cast<const v4u*>(src + (int64_t)i * cols));
    __builtin_amdgcn_sched_barrier(0);
    unsigned w[kPatchRows][2];
#pragma unroll
    for (int i = 0; i < kPatchRows; ++i) quantize8<FMT>(in[i], s, w[i][0], w[i][1]);
    uint8_t* dst = q + r0 * cols + c0;
#pragma unroll
    for (int i = 0; i < kPatchRows; ++i) store_hinted<STREAM>(v2u{w[i][0], w[i][1]}, reinterpret_cast<v2u*>(dst + (int64_t)i * cols));
    tile_stage_transposed(w, tr, tc, s_t);
    __syncthreads();
    // (qt_row_stride, qt_band_stride) = (rows, 128) for the transposed tensor as such, (128, cols x 128) in slabs
    tile_write_transposed(s_t, qt + (int64_t)bcol * kTileCols * qt_row_stride + (int64_t)brow * qt_band_stride, qt_row_stride);
}

// Everything else: tensors of few tiles, and ragged shapes of any size (plain transposed copy, or slabs where the shape
// has them; qt_row_stride, qt_band_stride as above), on the 64 x 128 tile.  The input is requested before a scale
// that has to be found from partial results, so that the two waits overlap.
// Measured against what was here before (one element per lane for shapes that are no multiples of 16 x 8; 16 x 8 patches
// without LDS for the others): 8100 x 5120 255 -> 35 us, 8112 x 5128 54 -> 38, 16000 x 9000 190 -> 174, 1777 x 960 14.7 -> 5.1.
// The 128 x 256 tile with the same guards took 39, 44 and 10.4 on the first, second and last.
template <int FMT>
__global__ __launch_bounds__(kTileThreads) void quantize_small_kernel(
    const uint16_t* __restrict__ x, int64_t rows, int64_t cols, const ScaleSource scale_src,
    uint8_t* __restrict__ q, uint8_t* __restrict__ qt, unsigned* __restrict__ zero_word, const SmallGrid grid,
    int64_t qt_row_stride, int64_t qt_band_stride) {
    __shared__ unsigned s_part[kTileThreads / kWave];
    __shared__ __attribute__((aligned(16))) uint8_t s_t[kSmallLdsBytes];
    if (zero_word && blockIdx.x == 0 && threadIdx.x == 0) *zero_word = 0u;
    unsigned brow, bcol;
    if (!small_tile(grid, brow, bcol)) return;
    int tr, tc;
    small_patch_origin(tr, tc);
    const int64_t R0 = (int64_t)brow * kSmallRows, C0 = (int64_t)bcol * kSmallCols, r0 = R0 + tr, c0 = C0 + tc;
    v4u in[kSmallPatch];
    float s = 0.0f;
    if (scale_src.partial == nullptr) s = *scale_src.d_scale;
    load_patch_upto(in, x + r0 * cols + c0, cols, rows - r0, cols - c0);
    if (scale_src.partial != nullptr) s = resolve_scale(scale_src, blockIdx.x == 0, s_part);
    unsigned w[kSmallPatch][2];
#pragma unroll
    for (int i = 0; i < kSmallPatch; ++i) quantize8<FMT>(in[i], s, w[i][0], w[i][1]);
    store_codes_upto(w, q + r0 * cols + c0, cols, rows - r0, cols - c0);
    small_stage_transposed(w, tr, tc, s_t);
    __syncthreads();
    small_write_transposed_upto(s_t, qt + C0 * qt_row_stride + (R0 / kTileRows) * qt_band_stride + R0 % kTileRows, qt_row_stride, rows - R0, cols - C0);
}

// No transposed copy wanted: the conversion is element-wise and the tensor can be taken as a flat array.  A
// workgroup converts kFlatUnits * 256 runs of 8 elements; load j of a wave covers 1 KB of contiguous input,
// its store 512 contiguous bytes (patches of rows, 64-byte pieces written, reached 4.8-5.2 TB/s where this reaches
// 5.9-6.1; with 1, 4 or 8 runs per lane instead of 2: 2-7 % less).
constexpr int kFlatUnits = 2;

template <int FMT>
__global__ __launch_bounds__(kQThreads) void quantize_flat_kernel(
    const uint16_t* __restrict__ x, int64_t n8, int n_tail, const ScaleSource scale_src, uint8_t* __restrict__ q,
    unsigned* __restrict__ zero_word) {
    __shared__ unsigned s_part[kQThreads / kWave];
    if (zero_word && blockIdx.x == 0 && threadIdx.x == 0) *zero_word = 0u;
    const float s = resolve_scale(scale_src, blockIdx.x == 0, s_part);
    const int64_t first = (int64_t)blockIdx.x * (kQThreads * kFlatUnits) + threadIdx.x;
    v4u in[kFlatUnits];
#pragma unroll
    for (int j = 0; j < kFlatUnits; ++j) {
        const int64_t u = first + j * kQThreads;
        if (u < n8) in[j] = __builtin_nontemporal_load(reinterpret_cast<const v4u*>(x) + u);
    }
#pragma unroll
    for (int j = 0; j < kFlatUnits; ++j) {
        const int64_t u = first + j * kQThreads;
        if (u < n8) {
            unsigned lo, hi;
            quantize8<FMT>(in[j], s, lo, hi);
            *(reinterpret_cast<v2u*>(q) + u) = v2u{lo, hi};
        }
    }
    if (blockIdx.x == 0 && (int)threadIdx.x < n_tail) {       // the n % 8 trailing elements
        const float p = __uint_as_float((unsigned)x[n8 * 8 + threadIdx.x] << 16) * s;
        q[n8 * 8 + threadIdx.x] = (uint8_t)(cvt_pair<FMT>(p, p, 0u, false) & 0xFFu);
    }
}

int launch_quantize(const void* x, int64_t rows, int64_t cols, const float* d_scale, int fmt,
                    uint8_t* q, uint8_t* q_t, unsigned* zero_word, hipStream_t stream, bool qt_slabs, bool read_next) {
    const ScaleSource src{d_scale, nullptr, 0, fp8_max(fmt), nullptr};
    return launch_quantize_from(x, rows, cols, src, fmt, q, q_t, zero_word, stream, qt_slabs, read_next);
}

bool quantize_can_write_slabs(int64_t rows, int64_t cols) {
    return tile_shape_ok(rows, cols);
}

int launch_quantize_from(const void* x, int64_t rows, int64_t cols, const ScaleSource& d_scale, int fmt,
                         uint8_t* q, uint8_t* q_t, unsigned* zero_word, hipStream_t stream, bool qt_slabs, bool read_next) {
    const uint16_t* xb = reinterpret_cast<const uint16_t*>(x);
    if (qt_slabs && !(q_t && quantize_can_write_slabs(rows, cols))) return -2;       // the caller asks first
    if (!q_t) {
        const int64_t n = rows * cols, n8 = n / 8;
        int64_t blocks = (n8 + kQThreads * kFlatUnits - 1) / (kQThreads * kFlatUnits);
        if (blocks < 1) blocks = 1;
        if (fmt == 0) hipLaunchKernelGGL((quantize_flat_kernel<0>), dim3((unsigned)blocks), dim3(kQThreads), 0, stream, xb, n8, (int)(n % 8), d_scale, q, zero_word);
        else hipLaunchKernelGGL((quantize_flat_kernel<1>), dim3((unsigned)blocks), dim3(kQThreads), 0, stream, xb, n8, (int)(n % 8), d_scale, q, zero_word);
    } else if (!takes_large_tile(rows, cols)) {
        const SmallGrid g = small_grid(rows, cols);
        const int64_t row_stride = qt_slabs ? kTileRows : rows, band_stride = qt_slabs ? cols * kTileRows : kTileRows;
        if (fmt == 0) hipLaunchKernelGGL((quantize_small_kernel<0>), dim3(g.blocks), dim3(kTileThreads), 0, stream, xb, rows, cols, d_scale, q, q_t, zero_word, g, row_stride, band_stride);
        else hipLaunchKernelGGL((quantize_small_kernel<1>), dim3(g.blocks), dim3(kTileThreads), 0, stream, xb, rows, cols, d_scale, q, q_t, zero_word, g, row_stride, band_stride);
    } else {
        const unsigned gc = (unsigned)(cols / kTileCols), gr = (unsigned)(rows / kTileRows);
        const int64_t row_stride = qt_slabs ? kTileRows : rows, band_stride = qt_slabs ? cols * kTileRows : kTileRows;
        auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3(gr * gc), dim3(kTileThreads), 0, stream, xb, cols, d_scale, q, q_t, zero_word, gc, row_stride, band_stride); };
        if (!read_next && streams_out(2 * rows * cols, 96)) { if (fmt == 0) launch(quantize_tile_kernel<0, true>); else launch(quantize_tile_kernel<1, true>); }
        else { if (fmt == 0) launch(quantize_tile_kernel<0, false>); else launch(quantize_tile_kernel<1, false>); }
    }
    return hipGetLastError() == hipSuccess ? 0 : -6;
}

}  // namespace llmq
