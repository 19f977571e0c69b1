// Host-side launchers of the gfx950 kernels (internal to the library; the public ABI is llmq.h).
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>
#include <stdlib.h>

namespace llmq {

// Tuning overrides come from the environment, for tests and tuning runs only: they are looked at when the
// process started with LLMQ_TUNING=1 (read once) and ignored otherwise, so the product path never calls
// getenv at launch.
inline const char* tuning_env(const char* name) {
    static const bool enabled = [] { const char* e = getenv("LLMQ_TUNING"); return e && e[0] == '1'; }();
    return enabled ? getenv(name) : nullptr;
}

// Workgroups of 256 lanes that one launch may have (fewer than 2^32 lanes, whole rounds of the 8 XCDs); what needs more is
// launched in pieces.  LLMQ_MAX_WORKGROUPS=n (tests): a smaller limit, a multiple of 8.
constexpr unsigned kMaxWorkgroups = (1u << 24) - 8;
inline unsigned max_workgroups() {
    if (const char* e = tuning_env("LLMQ_MAX_WORKGROUPS")) return (unsigned)atoi(e);
    return kMaxWorkgroups;
}

// The kernels that write FP8 codes in both layouts (quantize, and the SwiGLU and RMSNorm kernels that emit FP8 directly) work
// on tiles of 128 rows x 128 columns; a transposed copy in slabs is kept of tensors of 128-row x 256-column blocks.
constexpr int kTileRows = 128;
inline bool slab_shape_ok(int64_t rows, int64_t cols) { return rows % 128 == 0 && cols % 256 == 0; }

// Tensors of whole tiles take the tile kernels from about one tile per CU on, below that the 64 x 128 tile, of which there are
// twice as many; where the chip's next round of the large ones would be nearly empty, the small tile again.  Those with more to compute or to hold
// in registers have fewer workgroups resident and feel their rounds further up.  64 x 128 / 128 x 128 tile, microseconds, buffers of their own for every pass:
//   tiles                      256          320          384          512          540          640          720          960         1792         3584 (8192 x 7168)
//   quantize               5.6 /  5.3   6.3 /  6.3   6.8 /  6.7   8.0 /  7.8   9.5 /  9.2  10.4 / 10.2  11.5 / 10.9  15.3 / 14.4  29.6 / 24.4  51.3 / 38.0
//   RMSNorm codes          5.7 /  5.9   6.5 /  7.2   6.9 /  7.7   8.1 /  8.7   9.5 /  9.3  10.5 /  9.7  11.7 / 10.0  15.6 / 15.4  29.2 / 25.4  52.1 / 46.1
//     and the output       6.8 /  7.2   8.7 /  8.2   8.9 /  8.8  12.6 / 10.1  14.6 / 13.6  15.5 / 13.8  18.0 / 14.2  23.3 / 19.9
//   SwiGLU codes           8.7 /  8.4  10.3 / 11.8  10.7 / 12.2  12.9 / 13.3  14.2 / 15.9  14.7 / 16.4  16.8 / 16.7  21.9 / 20.3  41.0 / 35.2  75.4 / 68.1
//     and the output       9.8 /  9.6  11.2 / 12.7  11.8 / 13.1  14.1 / 14.0  18.2 / 17.8  19.3 / 18.2  22.1 / 19.5  29.0 / 26.9
//   RMSNorm codes beyond three resident workgroups per CU: 760 tiles 11.7 / 10.0, 770 11.9 / 12.9, 864 12.7 / 13.1, two sets of buffers in turn 960 14.2 / 14.8, 1008 14.7 /
//   15.2, 1053 15.4 / 15.6, 1092 16.0 / 15.8;  SwiGLU codes 680 16.3 / 16.5, 760 18.0 / 16.9;  with the output 392 13.4 / 13.2
// LLMQ_QUANT_TILE=0 / 1 (tests): always the one or, for shapes made of them, always the other.
struct LargeTiles {
    int64_t least;                              // the fewest tiles
    int64_t after, before;                      // ... but not for more than the one and less than the other
};
constexpr LargeTiles kQuantizeTiles{256, 0, 0}, kNormTiles{513, 768, 1024}, kNormOutputTiles{320, 0, 0}, kSwigluTiles{256, 256, 704}, kSwigluOutputTiles{256, 256, 392};
inline bool takes_large_tile(int64_t rows, int64_t cols, LargeTiles range) {
    if (rows % 128 != 0 || cols % 128 != 0) return false;
    if (const char* e = tuning_env("LLMQ_QUANT_TILE")) return atoi(e) != 0;
    const int64_t tiles = (rows / 128) * (cols / 128);
    return tiles >= range.least && (tiles <= range.after || tiles >= range.before);
}

// What the other tensors take when codes in both layouts are wanted:
//   kCodesElements  one element per lane: little code and short waits, so the fastest of all until there is something to move
//   kCodesNarrow    16 x 8 patches without LDS: up to 64 columns of whole patches (rows % 16 == 0, cols % 8 == 0)
//   kCodesSmall     the 64 x 128 tile
// Quantize kernel (the RMSNorm recompute kernels lie a few percent beside it), elements / patches / tile, microseconds:
//   narrow   16384 x 8 2.2 / 3.5 / 3.8, 60000 x 16 4.9 / 5.0 / 5.3, 1000000 x 16 42 / 27 / 41;  2048 x 64 2.9 / 3.2 / 3.8, 8000 x 64 5.0 / 3.3 / 4.0,
//            60000 x 32 9.5 / 4.6 / 6.1, 60000 x 64 23 / 5.4 / 6.7
//   whole patches, elements / tile   256 x 72 2.3 / 3.8, 2048 x 72 2.9 / 3.9, 2048 x 128 3.6 / 2.9, 8000 x 72 5.5 / 4.0
//   ragged rows   129 x 2056 3.3 / 3.6, 500 x 500 3.7 / 3.9, 300 x 701 3.5 / 3.8, 1000 x 333 4.2 / 4.0, 2001 x 200 4.6 / 3.5, 500 x 1001 5.1 / 3.9,
//            500 x 1000 4.9 / 4.2, 1000 x 1001 8.3 / 4.0, 4001 x 128 5.1 / 3.5, 4001 x 2730 62 / 12.8
//   few rows or columns leave most of the tile's lanes idle   7 x 300000 6.8 / 10.3, 33 x 20000 4.8 / 3.8, 20 x 50001 5.5 / 4.1, 200001 x 5 5.0 / 12.7,
//            16384 x 33 4.4 / 3.7, 60000 x 33 10.0 / 5.6, 60000 x 17 5.6 / 6.6, 200001 x 24 15.2 / 11.8
// LLMQ_CODES_KERNEL=0 / 1 / 2 (tests): the one, where it takes the shape.
enum CodesKind { kCodesElements, kCodesNarrow, kCodesSmall };
inline bool codes_narrow_ok(int64_t rows, int64_t cols) { return rows % 16 == 0 && cols % 8 == 0 && cols <= 64; }
inline CodesKind codes_kind(int64_t rows, int64_t cols) {
    const int64_t n = rows * cols;
    if (const char* e = tuning_env("LLMQ_CODES_KERNEL")) {
        const int k = atoi(e);
        if (k != kCodesNarrow || codes_narrow_ok(rows, cols)) return (CodesKind)k;
    }
    if (codes_narrow_ok(rows, cols)) return n < (cols <= 16 ? (int64_t)1 << 20 : (int64_t)5 << 16) ? kCodesElements : kCodesNarrow;
    if (rows % 16 == 0 && cols % 8 == 0) return n < ((int64_t)1 << 17) ? kCodesElements : kCodesSmall;
    const int64_t worth = (int64_t)3 << 17;
    if (rows < 8 || cols < (cols % 8 == 0 ? 24 : 32)) return kCodesElements;
    return n >= (rows < 16 ? 8 : rows < 32 || cols < 64 ? 2 : 1) * worth ? kCodesSmall : kCodesElements;
}

// Large results are stored with the streaming hint, so that they do not push out of the 256 MB memory-side cache what is
// still to be read.  Plain / streaming, passes over three sets of buffers in turn, and the same over one set (a first pass over
// buffers never touched before gains nothing: norm and recompute of 16384 x 5120 208 / 214): SwiGLU backward 8192 x 18944 (592 MiB of results)
// 283 / 267 us, forward 8192 x 18944 (296 MiB) 170 / 162, codes 8192 x 18944 197 / 187 (the row-major copy; the transposed
// one leaves in pieces of lines and stays plain); RMSNorm 16384 x 5120 (320 MiB) 134 / 127; codes in both layouts of
// 8192 x 7168 elements (112 MiB) 45.4 / 42.3, 4096 x 8192 (64 MiB) 26.1 / 26.2.  What the next kernel reads should stay in
// that cache when it fits: with results of 128 MiB streamed an MLP sub-block (4096 x 3072 x 8192) takes 1021 instead of 1013
// us.  Hence 144 MiB; 96 for the quantize calls of their own (a weight's codes are read much later); inside the linear
// calls, whose contraction reads the codes at once, codes are never streamed (no difference up to 32B-class layers).
// Only rows of whole 128-byte lines (cols_of_lines: columns a line holds): a line that two stores share goes to memory twice when it
// is streamed (backward of 60000 x 1000 131 / 177 us, of 1000000 x 72 193 / 275).
// LLMQ_STREAM=0 / 1 (tests): never, or for rows of whole lines always.
inline bool streams_out(int64_t result_bytes, int64_t cols, int64_t cols_of_line, int limit_mib = 144) {
    if (const char* e = tuning_env("LLMQ_STREAM")) return atoi(e) != 0 && cols % cols_of_line == 0;
    return cols % cols_of_line == 0 && result_bytes > ((int64_t)limit_mib << 20);
}

// Each returns 0 or LLMQ_ERR_DEVICE (-6).  Arguments are validated by the callers in api.hip.
constexpr int kAmaxMaxPartials = 1024;      // the absmax workspace holds one 32-bit word per block
int launch_amax(const void* x, size_t n, int fmt, float* d_amax, float* d_scale, void* ws,
                hipStream_t stream, int num_cus);
// The same with the partial results in the library's own file-scope device array (no workspace, no allocation).
int launch_amax_static(const void* x, size_t n, int fmt, float* d_amax, float* d_scale, hipStream_t stream,
                       int num_cus);
// Second stage of every absmax reduction: the maximum of n_partial BF16 magnitude patterns (one per
// workgroup of the first stage) becomes d_amax and, if d_scale is not NULL, the scale for fmt.
int launch_amax_final(const unsigned* partial, int n_partial, int fmt, float* d_amax, float* d_scale,
                      hipStream_t stream);
// BF16 x BF16 -> BF16 contraction without scales (T in elements), the baseline of the FP8 GEMM.
int launch_gemm_bf16_tn(const void* A, const void* B, int64_t R, int64_t C, int64_t T, void* c_bf16,
                        int accumulate, hipStream_t stream, int num_cus);
int launch_scale_from_amax(const float* d_amax, int fmt, float* d_scale, hipStream_t stream);
// Where a quantizing kernel gets its scale from: a scale on the device, or the per-workgroup results of
// the first stage of an absmax reduction over the same tensor, in which case every workgroup finishes the
// reduction itself (at most 1024 words) and the first one also stores the scale: the second-stage launch of
// the absmax is saved.
struct ScaleSource {
    const float* d_scale;        // used when partial == nullptr
    const unsigned* partial;     // BF16 magnitude patterns, one per workgroup of the first stage
    int n_partial;
    float fmax;                  // largest finite value of the target format
    float* d_scale_out;          // written (by one workgroup) when partial != nullptr
};

// One tensor to quantize.
//   zero_word: if not NULL, one 32-bit word the kernel also clears (the absmax accumulator of the GEMM
//     that follows in the same call, which saves a launch).
//   qt_slabs: the transposed copy is written in slabs of 128 contraction bytes (kLayoutSlabs of the contraction that
//     reads it: [cols, rows] with rows the contraction index); ask quantize_can_write_slabs() first (else -2).
// launch_quantize: a scale on the device, for the quantize calls of their own; launch_quantize_from: any source of the
// scale, for the operands of the linear calls, whose contraction reads the codes next (see streams_out).
int launch_quantize(const void* x, int64_t rows, int64_t cols, const float* d_scale, int fmt,
                    uint8_t* q, uint8_t* q_t, unsigned* zero_word, hipStream_t stream, bool qt_slabs);
int launch_quantize_from(const void* x, int64_t rows, int64_t cols, const ScaleSource& src, int fmt,
                         uint8_t* q, uint8_t* q_t, unsigned* zero_word, hipStream_t stream, bool qt_slabs);
struct QuantJob {
    const void* x;
    int64_t rows, cols;
    ScaleSource scale;
    uint8_t *q, *q_t;            // q_t may be NULL
    unsigned* zero_word;
    bool qt_slabs;
};
// launch_quantize_from for two tensors of the same format, in one launch where they take the same kernel.
int launch_quantize_pair(const QuantJob& first, const QuantJob& second, int fmt, hipStream_t stream);
bool quantize_can_write_slabs(int64_t rows, int64_t cols);
// First stage of the absmax only: one BF16 magnitude pattern per workgroup into partial; returns the number
// of workgroups (<= kAmaxMaxPartials) through n_partial.
int launch_amax_partial(const void* x, size_t n, unsigned* partial, int* n_partial, hipStream_t stream, int num_cus);
// The same for two tensors in one launch.
int launch_amax_partial_pair(const void* x, size_t n, unsigned* partial, int* n_partial, const void* x2, size_t n2, unsigned* partial2,
                             int* n_partial2, hipStream_t stream, int num_cus);
// Caller-owned device scratch for the binary32 pieces of output tiles whose contraction is shared among
// several workgroups (a ragged last round of tiles); {nullptr, 0}: every tile is computed by one workgroup.
struct GemmScratch {
    float* ptr;
    size_t bytes;
};
// What a contraction of this shape would use of it (0: nothing).
size_t gemm_scratch_bytes(int64_t R, int64_t C, int64_t T, int num_cus);
// How an operand [rows, T] of a contraction sits in memory: its rows of T contiguous bytes one after the other;
// the transposed tensor [T, rows]; or K step by K step ("slabs": byte (r, t) at (t / 128) rows 128 + r 128 + t % 128,
// T a multiple of 128), which is how the quantizer's tile kernel can write a transposed copy in contiguous pieces.
enum OperandLayout { kLayoutRows = 0, kLayoutTMajor = 1, kLayoutSlabs = 2 };
// Both operands kLayoutRows or kLayoutSlabs (slabs_a, slabs_b).
int launch_gemm_tn(const uint8_t* A, int fmtA, const uint8_t* B, int fmtB, int64_t R, int64_t C,
                   int64_t T, const float* d_scaleA, const float* d_scaleB, void* c_bf16,
                   int accumulate, float* d_amax_c, bool amax_is_zeroed, hipStream_t stream, int num_cus,
                   GemmScratch scratch, bool slabs_a = false, bool slabs_b = false);

// The 256 x 256 tile kernel with phase stamps: 16 words of 64 bits per workgroup id, gemm_phase_stamp_blocks() ids.
int gemm_phase_stamp_blocks(int64_t R, int64_t C);
int launch_gemm_phase_stamps(const uint8_t* A, const uint8_t* B, int64_t R, int64_t C, int64_t T, const float* sA,
                             const float* sB, void* c_bf16, float* d_amax_c, long long* stamps, int ieee_maximum,
                             hipStream_t stream, int num_cus);

// The same contraction with either operand in any OperandLayout: kLayoutTMajor: A is [T, R], B is [T, C] (the
// contraction index runs down the rows), so the backward GEMMs can read the untransposed quantized tensors.
int launch_gemm_fp8(const uint8_t* A, int fmtA, int layout_a, const uint8_t* B, int fmtB, int layout_b, int64_t R, int64_t C,
                    int64_t T, const float* d_scaleA, const float* d_scaleB, void* c_bf16, int accumulate,
                    float* d_amax_c, bool amax_is_zeroed, hipStream_t stream, int num_cus, GemmScratch scratch);

// SwiGLU with its extra outputs.  h, d_amax (with partial, the per-workgroup scratch), q and q_t are
// optional; q_fmt is only read when q is given.  swiglu_blocks() is the number of scratch words.
// qt_slabs (here and in the RMSNorm recompute launch): q_t in slabs of 128 contraction bytes, as in
// launch_quantize; needs q_t and slab_shape_ok(M, columns), else -2.
int64_t swiglu_blocks(int64_t M, int64_t I);
int launch_swiglu_fwd(const void* gu, int64_t M, int64_t I, void* h, unsigned* partial, int amax_fmt,
                      float* d_amax, float* d_scale, const float* d_qscale, int q_fmt, uint8_t* q, uint8_t* q_t,
                      hipStream_t stream, bool qt_slabs = false);
int launch_swiglu_bwd(const void* dh, const void* gu, int64_t M, int64_t I, void* dgu, unsigned* partial,
                      int amax_fmt, float* d_amax, float* d_scale, hipStream_t stream);

// RMSNorm + residual addition with absmax of the output (x, res_out optional together), and the
// element-wise recompute path that turns res, rstd and a known scale into FP8 codes (q_t, y optional).
// rmsnorm_blocks() is the number of scratch words of the forward launch.
int64_t rmsnorm_blocks(int64_t M);
int launch_rmsnorm_fwd(const void* res, const void* x, const void* w, int64_t M, int64_t C, float eps,
                       void* res_out, void* y, float* rstd, unsigned* partial, int fmt, float* d_amax,
                       float* d_scale, hipStream_t stream);
int launch_rmsnorm_apply_fp8(const void* res, const void* w, const float* rstd, int64_t M, int64_t C,
                             const float* d_qscale, int fmt, uint8_t* q, uint8_t* q_t, void* y, hipStream_t stream,
                             bool qt_slabs = false);

int launch_calibrate_mfma(int fmtA, int fmtB, int random_bits, int iters, float* d_sink, hipStream_t stream,
                          int num_cus);
int launch_calibrate_copy(const void* src, void* dst, size_t bytes, hipStream_t stream);

}  // namespace llmq
