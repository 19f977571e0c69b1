// Fused scale + FP8 cast + transposed copy (paper Section 3, kernel-fusion paragraph: quantization and
// transposition are one kernel; the FP8 GEMM wants both operands contraction-contiguous, so every
// quantized tensor is also needed transposed in the backward pass).
//
// HBM-bound: per element 2 bytes read, 1 byte written row-major and 1 byte written transposed.  A lane owns a patch of
// 8 rows x 8 columns (4 x 8 in tensors of few tiles): 16-byte loads, one binary32 multiply and the hardware RNE cast
// (clamped first, which makes it saturating), 8-byte stores of each row, a byte transpose in registers with byte
// permutes; the transposed patches leave through LDS in whole pieces of lines.
#include <stdlib.h>

#include "llmq_device.h"
#include "llmq_kernels.h"

namespace llmq {

constexpr int kQThreads = 256;

// One tensor of a launch.  Every kernel takes one (second.blocks == 0) or two, whose workgroups run side by side: the two
// operands of a forward pass then share a launch and its tail.
struct QuantTensor {
    const uint16_t* x;
    int64_t rows, cols;
    ScaleSource scale;
    uint8_t *q, *qt;
    unsigned* zero_word;
    // (qt_row_stride, qt_band_stride) = (rows, 128) for the transposed tensor as such, (128, cols x 128) in slabs
    int64_t qt_row_stride, qt_band_stride;
    SmallGrid grid;                              // 64 x 128 tiles
    unsigned blocks, first_block;                // of this launch (only the 64 x 128 tile and the flat kernel may need several)
};
struct QuantPair { QuantTensor first, second; };
__device__ inline const QuantTensor& tensor_of_block(const QuantPair& p, unsigned& block) {
    if (blockIdx.x < p.first.blocks) { block = blockIdx.x; return p.first; }
    block = blockIdx.x - p.first.blocks;
    return p.second;
}

// Tensors of at least 256 whole 128 x 128 tiles (the benchmark's tensors but for its smallest configuration's): full 128-byte
// lines on all three streams; the transposed patches go through LDS (the tile_* helpers, with what other tiles and lanes
// measured).  In slabs, against a tile of 128 x 256 with 16 rows per lane and lanes that follow each other stacked: 4096 x 3072 13.4 -> 10.6
// us, 8192 x 3584 26.4 -> 23.4 (5.0 TB/s), 8192 x 7168 42.4 -> 37.5 (6.3), 16384 x 5120 57.5 -> 51.8 (6.5); plain transposed copy 59.5 -> 52.8.
template <int FMT, bool STREAM>
__global__ __launch_bounds__(kTileThreads) void quantize_tile_kernel(const QuantPair pair) {
    __shared__ unsigned s_part[kTileThreads / kWave];
    __shared__ __attribute__((aligned(16))) uint8_t s_t[kTileLdsBytes];
    unsigned block;
    const QuantTensor& t = tensor_of_block(pair, block);
    if (t.zero_word && block == 0 && threadIdx.x == 0) *t.zero_word = 0u;
    // (the scale first: the conversions then follow the loads as they arrive; after them it costs 5 %)
    const float s = resolve_scale(t.scale, block == 0, s_part);
    const int64_t cols = t.cols;
    const unsigned grid_cols = (unsigned)(cols / kTileCols);
    const unsigned brow = block / grid_cols, bcol = block - brow * grid_cols;   // along the columns first
    int tr, tc;
    tile_patch_origin(tr, tc);
    const int64_t r0 = (int64_t)brow * kTileRows + tr, c0 = (int64_t)bcol * kTileCols + tc;
    v4u in[kPatchRows];
    const uint16_t* src = t.x + r0 * cols + c0;
#pragma unroll
    for (int i = 0; i < kPatchRows; ++i) in[i] = __builtin_nontemporal_load(reinterpret_cast<const v4u*>(src + (int64_t)i * cols));
    __builtin_amdgcn_sched_barrier(0);
    unsigned w[kPatchRows][2];
#pragma unroll
    for (int i = 0; i < kPatchRows; ++i) quantize8<FMT>(in[i], s, w[i][0], w[i][1]);
    uint8_t* dst = t.q + r0 * cols + c0;
#pragma unroll
    for (int i = 0; i < kPatchRows; ++i) store_hinted<STREAM>(v2u{w[i][0], w[i][1]}, reinterpret_cast<v2u*>(dst + (int64_t)i * cols));
    tile_stage_transposed(w, tr, tc, s_t);
    __syncthreads();
    tile_write_transposed(s_t, t.qt + (int64_t)bcol * kTileCols * t.qt_row_stride + (int64_t)brow * t.qt_band_stride, t.qt_row_stride);
}

// Tensors of few tiles, and ragged shapes with enough to move (plain transposed copy, or slabs where the shape
// has them), on the 64 x 128 tile.  The input is requested before a scale
// that has to be found from partial results, so that the two waits overlap.
// Measured against the kernels below (one element per lane for shapes that are no multiples of 16 x 8; 16 x 8 patches
// without LDS for the others): 8100 x 5120 255 -> 35 us, 8112 x 5128 54 -> 38, 16000 x 9000 190 -> 174, 1777 x 960 14.7 -> 5.1.
// The 128 x 256 tile with the same guards took 39, 44 and 10.4 on the first, second and last.
template <int FMT>
__global__ __launch_bounds__(kTileThreads) void quantize_small_kernel(const QuantPair pair) {
    __shared__ unsigned s_part[kTileThreads / kWave];
    __shared__ __attribute__((aligned(16))) uint8_t s_t[kSmallLdsBytes];
    unsigned block, brow, bcol;
    const QuantTensor& t = tensor_of_block(pair, block);
    block += t.first_block;
    if (t.zero_word && block == 0 && threadIdx.x == 0) *t.zero_word = 0u;
    if (!small_tile(t.grid, block, brow, bcol)) return;
    const int64_t rows = t.rows, cols = t.cols;
    int tr, tc;
    small_patch_origin(t.grid, tr, tc);
    const int64_t R0 = (int64_t)brow * kSmallRows, C0 = (int64_t)bcol * kSmallCols, r0 = R0 + tr, c0 = C0 + tc;
    v4u in[kSmallPatch];
    float s = 0.0f;
    if (t.scale.partial == nullptr) s = *t.scale.d_scale;
    load_patch_upto(in, t.x + r0 * cols + c0, cols, c0, rows - r0, cols - c0);
    if (t.scale.partial != nullptr) s = resolve_scale(t.scale, block == 0, s_part);
    unsigned w[kSmallPatch][2];
#pragma unroll
    for (int i = 0; i < kSmallPatch; ++i) quantize8<FMT>(in[i], s, w[i][0], w[i][1]);
    store_codes_upto(w, t.q + r0 * cols + c0, cols, rows - r0, cols - c0);
    small_stage_transposed(w, tr, tc, s_t);
    __syncthreads();
    small_write_transposed_upto(s_t, t.qt + C0 * t.qt_row_stride + (R0 / kTileRows) * t.qt_band_stride + R0 % kTileRows, t.qt_row_stride, rows - R0, cols - C0);
}

// Narrow tensors of whole 16 x 8 patches, which would leave most lanes of the 64 x 128 tile idle (codes_kind).
template <int FMT>
__global__ __launch_bounds__(kQThreads) void quantize_narrow_kernel(const QuantPair pair) {
    __shared__ unsigned s_part[kQThreads / kWave];
    unsigned block;
    const QuantTensor& t = tensor_of_block(pair, block);
    if (t.zero_word && block == 0 && threadIdx.x == 0) *t.zero_word = 0u;
    const float s = resolve_scale(t.scale, block == 0, s_part);          // before any lane leaves
    const int64_t rows = t.rows, cols = t.cols;
    int tr, tc;
    narrow_patch_origin(tr, tc);
    const int64_t r0 = (int64_t)block * kNarrowRows + tr;
    if (r0 >= rows || tc >= cols) return;
    const uint16_t* src = t.x + r0 * cols + tc;
    v4u in[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) in[i] = __builtin_nontemporal_load(reinterpret_cast<const v4u*>(src + (int64_t)i * cols));
    __builtin_amdgcn_sched_barrier(0);
    unsigned w[16][2];
#pragma unroll
    for (int i = 0; i < 16; ++i) quantize8<FMT>(in[i], s, w[i][0], w[i][1]);
    uint8_t* dst = t.q + r0 * cols + tc;
#pragma unroll
    for (int i = 0; i < 16; ++i) *reinterpret_cast<v2u*>(dst + (int64_t)i * cols) = v2u{w[i][0], w[i][1]};
    narrow_write_transposed(w, t.qt + (int64_t)tc * rows + r0, rows);
}

// One element per lane: small tensors, and ragged ones of few rows or columns (codes_kind).
constexpr int64_t kElementsMaxBlocks = 65536;
template <int FMT>
__global__ __launch_bounds__(kQThreads) void quantize_elements_kernel(const QuantPair pair) {
    __shared__ unsigned s_part[kQThreads / kWave];
    unsigned block;
    const QuantTensor& t = tensor_of_block(pair, block);
    if (t.zero_word && block == 0 && threadIdx.x == 0) *t.zero_word = 0u;
    const float s = resolve_scale(t.scale, block == 0, s_part);
    const int64_t rows = t.rows, cols = t.cols, n = rows * cols;
    for (int64_t i = (int64_t)block * kQThreads + threadIdx.x; i < n; i += (int64_t)t.blocks * kQThreads) {
        const float p = __uint_as_float((unsigned)t.x[i] << 16) * s;
        const uint8_t code = (uint8_t)(cvt_pair<FMT>(p, p, 0u, false) & 0xFFu);
        t.q[i] = code;
        const int64_t r = i / cols, c = i - r * cols;
        t.qt[c * rows + r] = code;
    }
}

// No transposed copy wanted: the conversion is element-wise and the tensor can be taken as a flat array.  A
// workgroup converts kFlatUnits * 256 runs of 8 elements; load j of a wave covers 1 KB of contiguous input,
// its store 512 contiguous bytes (patches of rows, 64-byte pieces written, reached 4.8-5.2 TB/s where this reaches
// 5.9-6.1; with 1, 4 or 8 runs per lane instead of 2: 2-7 % less).
constexpr int kFlatUnits = 2;

template <int FMT>
__global__ __launch_bounds__(kQThreads) void quantize_flat_kernel(const QuantPair pair) {
    __shared__ unsigned s_part[kQThreads / kWave];
    unsigned block;
    const QuantTensor& t = tensor_of_block(pair, block);
    block += t.first_block;
    if (t.zero_word && block == 0 && threadIdx.x == 0) *t.zero_word = 0u;
    const float s = resolve_scale(t.scale, block == 0, s_part);
    const int64_t n = t.rows * t.cols, n8 = n / 8;
    const int64_t first = (int64_t)block * (kQThreads * kFlatUnits) + threadIdx.x;
    v4u in[kFlatUnits];
#pragma unroll
    for (int j = 0; j < kFlatUnits; ++j) {
        const int64_t u = first + j * kQThreads;
        if (u < n8) in[j] = __builtin_nontemporal_load(reinterpret_cast<const v4u*>(t.x) + u);
    }
#pragma unroll
    for (int j = 0; j < kFlatUnits; ++j) {
        const int64_t u = first + j * kQThreads;
        if (u < n8) {
            unsigned lo, hi;
            quantize8<FMT>(in[j], s, lo, hi);
            *(reinterpret_cast<v2u*>(t.q) + u) = v2u{lo, hi};
        }
    }
    if (block == 0 && (int)threadIdx.x < (int)(n % 8)) {       // the n % 8 trailing elements
        const float p = __uint_as_float((unsigned)t.x[n8 * 8 + threadIdx.x] << 16) * s;
        t.q[n8 * 8 + threadIdx.x] = (uint8_t)(cvt_pair<FMT>(p, p, 0u, false) & 0xFFu);
    }
}

bool quantize_can_write_slabs(int64_t rows, int64_t cols) { return slab_shape_ok(rows, cols); }

// Which kernel a tensor takes, and what the kernel is told about it
enum QuantKind { kQuantFlat, kQuantElements, kQuantNarrow, kQuantSmall, kQuantTile };
static QuantKind quant_kind(const QuantJob& j) {
    if (!j.q_t) return kQuantFlat;
    if (takes_large_tile(j.rows, j.cols, kQuantizeTiles)) return kQuantTile;
    if (j.qt_slabs) return kQuantSmall;
    const CodesKind k = codes_kind(j.rows, j.cols);
    return k == kCodesElements ? kQuantElements : k == kCodesNarrow ? kQuantNarrow : kQuantSmall;
}

static QuantTensor quant_tensor(const QuantJob& j, QuantKind kind) {
    QuantTensor t{};
    t.x = reinterpret_cast<const uint16_t*>(j.x);
    t.rows = j.rows; t.cols = j.cols; t.scale = j.scale; t.q = j.q; t.qt = j.q_t; t.zero_word = j.zero_word;
    t.qt_row_stride = j.qt_slabs ? kTileRows : j.rows;
    t.qt_band_stride = j.qt_slabs ? j.cols * kTileRows : kTileRows;
    if (kind == kQuantFlat) {
        const int64_t n8 = j.rows * j.cols / 8, blocks = (n8 + kQThreads * kFlatUnits - 1) / (kQThreads * kFlatUnits);
        t.blocks = blocks < 1 ? 1u : (unsigned)blocks;
    } else if (kind == kQuantElements) {
        const int64_t blocks = (j.rows * j.cols + kQThreads - 1) / kQThreads;
        t.blocks = (unsigned)(blocks < kElementsMaxBlocks ? blocks : kElementsMaxBlocks);
    } else if (kind == kQuantNarrow) {
        t.blocks = (unsigned)((j.rows + kNarrowRows - 1) / kNarrowRows);
    } else if (kind == kQuantTile) {
        t.blocks = (unsigned)((j.rows / kTileRows) * (j.cols / kTileCols));
    } else {
        t.grid = small_grid(j.rows, j.cols, true, true);
        t.blocks = t.grid.blocks;
    }
    return t;
}

template <int FMT>
static void launch_kind(QuantKind kind, const QuantPair& pair, bool stream_out, hipStream_t stream) {
    auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, dim3(pair.first.blocks + pair.second.blocks), dim3(kQThreads), 0, stream, pair); };
    if (kind == kQuantFlat) launch(quantize_flat_kernel<FMT>);
    else if (kind == kQuantElements) launch(quantize_elements_kernel<FMT>);
    else if (kind == kQuantNarrow) launch(quantize_narrow_kernel<FMT>);
    else if (kind == kQuantSmall) launch(quantize_small_kernel<FMT>);
    else if (stream_out) launch(quantize_tile_kernel<FMT, true>);
    else launch(quantize_tile_kernel<FMT, false>);
}

// second: another tensor of the same format, or NULL.  Tensors that take the same kernel share a launch.
static int launch_jobs(const QuantJob& first, const QuantJob* second, int fmt, bool read_next, hipStream_t stream) {
    for (const QuantJob* j : {&first, second})
        if (j && j->qt_slabs && !(j->q_t && quantize_can_write_slabs(j->rows, j->cols))) return -2;       // the caller asks first
    const unsigned most = max_workgroups();
    auto launch = [&](const QuantTensor& t, const QuantTensor& with, QuantKind kind) {
        const QuantPair pair{t, with};
        const bool stream_out = !read_next && streams_out(2 * t.rows * t.cols, t.cols, 128, 96);
        if (fmt == 0) launch_kind<0>(kind, pair, stream_out, stream);
        else launch_kind<1>(kind, pair, stream_out, stream);
    };
    auto launch_one = [&](QuantTensor t, QuantKind kind) {                       // in pieces, if it has to be
        for (unsigned blocks = t.blocks; t.first_block < blocks; t.first_block += most) {
            t.blocks = blocks - t.first_block < most ? blocks - t.first_block : most;
            launch(t, QuantTensor{}, kind);
        }
    };
    QuantKind kind = quant_kind(first), kind2 = second ? quant_kind(*second) : kind;
    // (the 64 x 128 tile takes every shape: one launch of both on it beats two launches)
    if ((kind == kQuantElements && kind2 == kQuantSmall) || (kind == kQuantSmall && kind2 == kQuantElements)) kind = kind2 = kQuantSmall;
    const QuantTensor t = quant_tensor(first, kind), t2 = second ? quant_tensor(*second, kind2) : QuantTensor{};
    if (second && kind == kind2 && t.blocks < most && t2.blocks < most - t.blocks) {
        launch(t, t2, kind);
    } else {
        launch_one(t, kind);
        if (second) launch_one(t2, kind2);
    }
    return hipGetLastError() == hipSuccess ? 0 : -6;
}

int launch_quantize(const void* x, int64_t rows, int64_t cols, const float* d_scale, int fmt,
                    uint8_t* q, uint8_t* q_t, unsigned* zero_word, hipStream_t stream, bool qt_slabs) {
    const ScaleSource src{d_scale, nullptr, 0, fp8_max(fmt), nullptr};
    return launch_jobs(QuantJob{x, rows, cols, src, q, q_t, zero_word, qt_slabs}, nullptr, fmt, false, stream);
}

int launch_quantize_from(const void* x, int64_t rows, int64_t cols, const ScaleSource& src, int fmt,
                         uint8_t* q, uint8_t* q_t, unsigned* zero_word, hipStream_t stream, bool qt_slabs) {
    return launch_jobs(QuantJob{x, rows, cols, src, q, q_t, zero_word, qt_slabs}, nullptr, fmt, true, stream);
}

int launch_quantize_pair(const QuantJob& first, const QuantJob& second, int fmt, hipStream_t stream) {
    return launch_jobs(first, &second, fmt, true, stream);
}

}  // namespace llmq
