// FP8 contraction with both operands contraction-contiguous ("TN"), its BF16 baseline, and the kernels for
// shapes no tuned tile divides.  The tile kernel itself is in gemm_tile.h.
#include "gemm_tile.h"

namespace llmq {

void launch_gemm_generic(const uint8_t* A, int fmtA, int layout_a, const uint8_t* B, int fmtB, int layout_b, int64_t R, int64_t C,
                         int64_t T, const float* sA, const float* sB, void* c, int accumulate, unsigned* amax,
                         hipStream_t stream);

// ---- generic kernel: one wavefront per 16x16 outputs, v_mfma_f32_16x16x128_f8f6f4, guarded loads.
// ta / tb: the operand's OperandLayout; the bytes of a T-major operand ([T, R] or [T, Cn]) are gathered one by one.
template <int FA, int FB>
__global__ __launch_bounds__(256) void gemm_generic_kernel(
    const uint8_t* __restrict__ A, const uint8_t* __restrict__ B, uint16_t* __restrict__ C,
    int64_t R, int64_t Cn, int64_t T, const float* __restrict__ d_sA, const float* __restrict__ d_sB,
    int accumulate, unsigned* __restrict__ amax_bits, int ta, int tb) {
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = threadIdx.x / kWave;
    const int64_t r0 = ((int64_t)blockIdx.y * 2 + (wave >> 1)) * 16;
    const int64_t c0 = ((int64_t)blockIdx.x * 2 + (wave & 1)) * 16;
    const int64_t ar = r0 + (lane & 15), bc = c0 + (lane & 15);
    const bool a_ok = ar < R, b_ok = bc < Cn;
    const bool vec_ok = (T % 16) == 0;
    auto load32 = [&](const uint8_t* base, bool ok, int64_t row, int64_t k, int tmajor, int64_t ld) -> v8i {
        v8i v = {0, 0, 0, 0, 0, 0, 0, 0};
        if (!ok || k >= T) return v;
        if (tmajor == kLayoutSlabs) {                 // 32 contiguous bytes of the row's K step (T % 128 == 0)
            const uint8_t* p = base + (k >> 7) * (ld * 128) + row * 128 + (k & 127);
            v4i lo = *reinterpret_cast<const v4i*>(p), hi = *reinterpret_cast<const v4i*>(p + 16);
            return v8i{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        }
        if (tmajor) {
            for (int w = 0; w < 8; ++w) {
                unsigned word = 0;
                for (int e = 0; e < 4; ++e) {
                    int64_t kk = k + w * 4 + e;
                    if (kk < T) word |= (unsigned)base[kk * ld + row] << (8 * e);
                }
                v[w] = (int)word;
            }
            return v;
        }
        const uint8_t* p = base + row * T + k;
        if (vec_ok && k + 32 <= T) {
            v4i lo = *reinterpret_cast<const v4i*>(p), hi = *reinterpret_cast<const v4i*>(p + 16);
            return v8i{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
        }
        for (int w = 0; w < 8; ++w) {
            unsigned word = 0;
            for (int e = 0; e < 4; ++e) {
                int64_t kk = k + w * 4 + e;
                if (kk < T) word |= (unsigned)p[w * 4 + e] << (8 * e);   // beyond T: code 0x00 = +0
            }
            v[w] = (int)word;
        }
        return v;
    };
    v4f acc = {0.0f, 0.0f, 0.0f, 0.0f};
    for (int64_t k0 = 0; k0 < T; k0 += 128) {
        const int64_t k = k0 + (lane >> 4) * 32;
        v8i a = load32(A, a_ok, ar, k, ta, R);
        v8i b = load32(B, b_ok, bc, k, tb, Cn);
        acc = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(b, a, acc, FB, FA, 0, 0, 0, 0);
    }
    // lane holds row r0 + lane % 16, columns c0 + 4 * (lane / 16) + 0..3
    // de-scaled as the tile kernels do it, so that the same sums give the same bytes whichever kernel ran
    const float inv_a = 1.0f / *d_sA, inv_b = 1.0f / *d_sB, inv_ab = inv_a * inv_b;
    const bool one_mul = inv_ab >= 1.17549435e-38f && inv_ab <= 3.402823466e+38f;
    const float m1 = one_mul ? inv_ab : inv_a, m2 = one_mul ? 1.0f : inv_b;
    unsigned mag = 0;
    const int64_t r = r0 + (lane & 15);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        const int64_t c = c0 + (lane >> 4) * 4 + e;
        if (r < R && c < Cn) {
            float y = acc[e] * m1 * m2;
            uint16_t* dst = C + r * Cn + c;
            if (accumulate) y += __uint_as_float((unsigned)*dst << 16);
            __bf16 o = (__bf16)y;
            unsigned bits = __builtin_bit_cast(uint16_t, o);
            *dst = (uint16_t)bits;
            bits &= 0x7FFFu;
            mag = mag > bits ? mag : bits;
        }
    }
    if (amax_bits) {
        mag = wave_max_u32(mag);
        if (lane == 0) atomicMax(amax_bits, amax_bits_from_bf16_mag(mag));
    }
}

// ---- Few outputs: tiles of 64 x 64 or 32 x 32.
//
// What a CU reads per K step sets the pace of a problem that has fewer tiles than the chip has CUs: a 128 x 128 tile takes 32 KB and
// 0.29 us, and the rest of the chip looks on.  Here a workgroup of four waves (2 x 2) has a tile of SIDE x SIDE, 16 or 8 KB a
// step.  Four K steps make a stage: one wait and two barriers for all four, and 64 (SIDE 64: two stages) or 96 KB (SIDE 32: four) on
// their way while one is multiplied.  Slabs, swizzle and fragments are those of the tile kernel; the sums have its order, so the bytes are
// the same.  Operands in rows of whole 16-byte chunks, or in slabs; what lies behind an operand or the end of a row arrives
// as zeros (offsets beyond the buffer's range).
constexpr int kMiniSteps = 4;                                            // K steps of a stage
template <int FA, int FB, int SIDE>
__global__ __launch_bounds__(kGemmThreads, 1) void gemm_mini_kernel(
    const uint8_t* __restrict__ A, const uint8_t* __restrict__ B, uint16_t* __restrict__ C, int R, int Cn, int T,
    const float* __restrict__ d_sA, const float* __restrict__ d_sB, int accumulate, unsigned* __restrict__ amax_bits, int ldA, int ldB, int ksA, int ksB,
    int tiles_r, int n_tiles) {
    constexpr int kOutOfRange = 0x7FFFFF00;
    constexpr int kSlab = SIDE * BK, kOperand = kMiniSteps * kSlab;      // bytes of one operand in a K step, in a stage
    constexpr int ST = SIDE == 64 ? 2 : 4, NB = SIDE / 32;               // stages; blocks of 16 x 16 per wave and side
    // one LDS object per stage and operand or per stage, which the compiler tells apart (see the tile kernel)
    __shared__ __attribute__((aligned(1024))) uint8_t s_0[32768];
    __shared__ __attribute__((aligned(1024))) uint8_t s_1[32768];
    __shared__ __attribute__((aligned(1024))) uint8_t s_2[32768];
    __shared__ __attribute__((aligned(1024))) uint8_t s_3[32768];
    static_assert(ST * 2 * kOperand == 4 * 32768, "");
    const int pos = walk_position(blockIdx.x, n_tiles);
    if (pos < 0) return;
    const int tc = pos / tiles_r, tr = pos - tc * tiles_r;               // down the rows: neighbours share the columns' operand
    const int lane = threadIdx.x & (kWave - 1), wave = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave);
    const int r0 = tr * SIDE, c0 = tc * SIDE;
    const float scale_a = FA == kFmtBf16 ? 1.0f : *d_sA, scale_b = FB == kFmtBf16 ? 1.0f : *d_sB;
    const int nk = (T + BK - 1) / BK, ns = (nk + kMiniSteps - 1) / kMiniSteps;
    auto range = [&](int rows_left, int ld, int ks) -> unsigned {
        const int n = rows_left < SIDE ? rows_left : SIDE;
        return ks == BK ? (unsigned)((size_t)(n - 1) * ld + T) : (unsigned)((size_t)(T / BK - 1) * ks + (size_t)(n - 1) * ld + BK);
    };
    const __amdgpu_buffer_rsrc_t rsA = make_rsrc(A + (size_t)r0 * ldA, range(R - r0, ldA, ksA));
    const __amdgpu_buffer_rsrc_t rsB = make_rsrc(B + (size_t)c0 * ldB, range(Cn - c0, ldB, ksB));
    // Loads: an instruction moves 8 rows x 128 bytes; the wave's rows are [SIDE / 4 wave, SIDE / 4 (wave + 1))
    constexpr int kPerSlab = SIDE / 32, kLoads = 2 * kMiniSteps * kPerSlab;
    const int ld_row = lane >> 3;
    auto issue_stage = [&](uint8_t* bufA, uint8_t* bufB, int stage) {
#pragma unroll
        for (int j = 0; j < kMiniSteps; ++j) {
            const int step = stage * kMiniSteps + j;
#pragma unroll
            for (int m = 0; m < kPerSlab; ++m) {
                const int row = wave * (SIDE / 4) + 8 * m + ld_row;      // its index modulo 16 sets the swizzle
                const int chunk = ((lane & 7) ^ row_swizzle(row & 15)) << 4;
                const bool there = step < nk && step * BK + chunk < T;   // (T % 16 == 0: a chunk exists or not)
                const int offA = there ? row * ldA + chunk + (int)((unsigned)step * (unsigned)ksA) : kOutOfRange;
                const int offB = there ? row * ldB + chunk + (int)((unsigned)step * (unsigned)ksB) : kOutOfRange;
                const int dst = j * kSlab + (wave * (SIDE / 4) + 8 * m) * BK;
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rsA, (lds_void*)(bufA + dst), 16, offA, 0, 0, 0);
                __builtin_amdgcn_raw_ptr_buffer_load_lds(rsB, (lds_void*)(bufB + dst), 16, offB, 0, 0, 0);
            }
        }
    };
    const int wr = wave >> 1, wc = wave & 1;
    const int fr_row = lane & 15, fr_q = lane >> 4, swz = row_swizzle(fr_row);
    const int ch0 = ((fr_q * 2) ^ swz) << 4, ch1 = ((fr_q * 2 + 1) ^ swz) << 4;
    auto fragment = [&](const uint8_t* slab, int first_row) -> v8i {
        const uint8_t* p = slab + (first_row + fr_row) * BK;
        const v4i lo = *reinterpret_cast<const v4i*>(p + ch0), hi = *reinterpret_cast<const v4i*>(p + ch1);
        return v8i{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]};
    };
    v4f acc[NB][NB];
#pragma unroll
    for (int i = 0; i < NB; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) acc[i][j] = v4f{0.0f, 0.0f, 0.0f, 0.0f};
    auto stage_step = [&](uint8_t* bufA, uint8_t* bufB, int stage) __attribute__((always_inline)) {
        wait_vmcnt<(ST - 1) * kLoads>();                                 // this stage has landed, the later ones are on their way
        lds_barrier_in_flight();
        v8i a[kMiniSteps][NB], b[kMiniSteps][NB];
#pragma unroll
        for (int j = 0; j < kMiniSteps; ++j)
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                a[j][i] = fragment(bufA + j * kSlab, wr * 16 * NB + 16 * i);
                b[j][i] = fragment(bufB + j * kSlab, wc * 16 * NB + 16 * i);
            }
#pragma unroll
        for (int j = 0; j < kMiniSteps; ++j)
#pragma unroll
            for (int i = 0; i < NB; ++i)
#pragma unroll
                for (int k = 0; k < NB; ++k) {
                    if constexpr (FA == kFmtBf16) {
                        const v8i &x = b[j][k], &y = a[j][i];
                        const v4i x0 = {x[0], x[1], x[2], x[3]}, x1 = {x[4], x[5], x[6], x[7]}, y0 = {y[0], y[1], y[2], y[3]}, y1 = {y[4], y[5], y[6], y[7]};
                        acc[i][k] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, x0), __builtin_bit_cast(bf16x8, y0), acc[i][k], 0, 0, 0);
                        acc[i][k] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, x1), __builtin_bit_cast(bf16x8, y1), acc[i][k], 0, 0, 0);
                    } else {
                        acc[i][k] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(b[j][k], a[j][i], acc[i][k], FB, FA, 0, 0, 0, 0);
                    }
                }
        lds_barrier_in_flight();                                         // everybody has read the stage: it may be overwritten
        issue_stage(bufA, bufB, stage + ST);                             // (beyond the last stage: nothing is fetched, zeros are written)
    };
    auto half = [&](uint8_t* buf) { return SIDE == 64 ? buf : buf + kOperand; };
    if constexpr (SIDE == 64) {
        issue_stage(s_0, s_1, 0);
        issue_stage(s_2, s_3, 1);
        int st = 0;
        for (; st + 1 < ns; st += 2) {                                   // (the same order of loads on every way round: the compiler counts them)
            stage_step(s_0, s_1, st);
            stage_step(s_2, s_3, st + 1);
        }
        if (st < ns) stage_step(s_0, s_1, st);
    } else {
        issue_stage(s_0, half(s_0), 0);
        issue_stage(s_1, half(s_1), 1);
        issue_stage(s_2, half(s_2), 2);
        issue_stage(s_3, half(s_3), 3);
        int st = 0;
        for (; st + 3 < ns; st += 4) {
            stage_step(s_0, half(s_0), st);
            stage_step(s_1, half(s_1), st + 1);
            stage_step(s_2, half(s_2), st + 2);
            stage_step(s_3, half(s_3), st + 3);
        }
        if (st < ns) stage_step(s_0, half(s_0), st);
        if (st + 1 < ns) stage_step(s_1, half(s_1), st + 1);
        if (st + 2 < ns) stage_step(s_2, half(s_2), st + 2);
    }
    wait_vmcnt<0>();                                                     // nothing lands in LDS behind the workgroup's end
    const float inv_a = 1.0f / scale_a, inv_b = 1.0f / scale_b, inv_ab = inv_a * inv_b;
    const bool one_mul = inv_ab >= 1.17549435e-38f && inv_ab <= 3.402823466e+38f;
    const float m1 = one_mul ? inv_ab : inv_a, m2 = one_mul ? 1.0f : inv_b;
    const bool vector = Cn % 4 == 0;
    unsigned mag = 0;
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int r = r0 + wr * 16 * NB + 16 * i + (lane & 15);
#pragma unroll
        for (int k = 0; k < NB; ++k) {
            const int c = c0 + wc * 16 * NB + 16 * k + (lane >> 4) * 4;
            if (r >= R || c >= Cn) continue;
            uint16_t* dst = C + (size_t)r * Cn + c;
            const int valid = Cn - c;
            uint16_t old[4] = {0, 0, 0, 0}, out[4];
            if (accumulate) {
                if (vector) {
                    const v2u o = *reinterpret_cast<const v2u*>(dst);
                    old[0] = (uint16_t)o[0]; old[1] = (uint16_t)(o[0] >> 16); old[2] = (uint16_t)o[1]; old[3] = (uint16_t)(o[1] >> 16);
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) if (e < valid) old[e] = dst[e];
                }
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                float y = acc[i][k][e] * m1 * m2;
                if (accumulate) y += __uint_as_float((unsigned)old[e] << 16);
                out[e] = __builtin_bit_cast(uint16_t, (__bf16)y);
                const unsigned m = out[e] & 0x7FFFu;
                if (e < valid) mag = mag > m ? mag : m;
            }
            if (vector) *reinterpret_cast<v2u*>(dst) = v2u{out[0] | (unsigned)out[1] << 16, out[2] | (unsigned)out[3] << 16};
            else {
#pragma unroll
                for (int e = 0; e < 4; ++e) if (e < valid) dst[e] = out[e];
            }
        }
    }
    if (amax_bits) {
        __syncthreads();
        mag = block_max_u32<kGemmThreads>(mag, reinterpret_cast<unsigned*>(s_0));
        if (threadIdx.x == 0) {
            const unsigned bits = amax_bits_from_bf16_mag(mag);
            if (bits > __hip_atomic_load(amax_bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) atomicMax(amax_bits, bits);
        }
    }
}

// BF16 operands, any shape: one output element per lane and trip, binary32 accumulation along t.
__global__ __launch_bounds__(256) void gemm_bf16_generic_kernel(
    const uint16_t* __restrict__ A, const uint16_t* __restrict__ B, uint16_t* __restrict__ C,
    int64_t R, int64_t Cn, int64_t T, int accumulate) {
    const int64_t n = R * Cn;
    for (int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; idx < n; idx += (int64_t)gridDim.x * blockDim.x) {
        const int64_t r = idx / Cn, c = idx - r * Cn;
        float acc = 0.0f;
        for (int64_t t = 0; t < T; ++t)
            acc = __builtin_fmaf(__uint_as_float((unsigned)A[r * T + t] << 16), __uint_as_float((unsigned)B[c * T + t] << 16), acc);
        if (accumulate) acc += __uint_as_float((unsigned)C[idx] << 16);
        C[idx] = __builtin_bit_cast(uint16_t, (__bf16)acc);
    }
}

__global__ void gemm_amax_reset_kernel(unsigned* amax_bits) {
    if (threadIdx.x == 0 && blockIdx.x == 0) *amax_bits = 0u;
}

// ---- host side: tile choice and launch

// Picks the wave tile NI x NJ (workgroup tile 64 NI x 64 NJ) that finishes soonest under a simple
// model: every CU works through its share of the tiles, a tile costs NI * NJ MFMA blocks per K step
// divided by the measured efficiency of that shape relative to 4 x 4 (smaller tiles read more LDS
// and L2 bytes per MFMA; 2 x 2 tiles fit two workgroups per CU, which hide each other's stalls).
TileChoice choose_tile(int64_t R, int64_t C, int64_t T, int num_cus, size_t scratch_bytes, bool bf16) {
    static const float eff[5][5] = {{0, 0, 0, 0, 0}, {0, 0, 0, 0, 0}, {0, 0, 0.90f, 0.74f, 0.77f},
                                    {0, 0, 0.74f, 0.70f, 0.83f}, {0, 0, 0.77f, 0.83f, 1.00f}};
    TileChoice best{0, 0};
    if (T % BK != 0 || T >= (1ll << 23)) return best;
    // Override for tests and tuning: LLMQ_GEMM_TILE=IxJ forces that wave tile where it divides the problem.
    if (const char* force = tuning_env("LLMQ_GEMM_TILE")) {
        const int ni = force[0] - '0', nj = force[0] && force[1] ? force[2] - '0' : 0;
        if (ni >= 2 && ni <= 4 && nj >= 2 && nj <= 4 && R % (64 * ni) == 0 && C % (64 * nj) == 0) return TileChoice{ni, nj};
    }
    // At most one 128 x 128 tile per CU: that tile, with four LDS stages, whatever the model says about larger ones (1024 x
    // 3072 x 3072: 14.6 us against 18.0 with 192 x 128 tiles; 128 x 9984 x 13184: 68 against 98).  Contractions long enough
    // for sharing out tiles keep the model's choice when there is scratch for it.
    if (R % 128 == 0 && C % 128 == 0 && (scratch_bytes == 0 || T / BK < 64) &&
        (R / 128) * (C / 128) <= resident_slots(num_cus, 2, 2) / 2)
        return TileChoice{2, 2};
    double best_cost = 0;
    for (int ni = 4; ni >= 2; --ni)
        for (int nj = 4; nj >= 2; --nj) {
            if (R % (64 * ni) != 0 || C % (64 * nj) != 0) continue;
            const int64_t tiles = (R / (64 * ni)) * (C / (64 * nj));
            if (tiles >= (1ll << 30)) continue;
            const int per_cu = (ni == 2 && nj == 2) ? 2 : 1;          // workgroups resident per CU
            const int64_t slots = resident_slots(num_cus, ni, nj);
            const int64_t rounds = (tiles + slots - 1) / slots;
            // two resident 2 x 2 workgroups overlap each other's prologue and epilogue, which pays most
            // when the contraction is short
            // (BF16 moves twice the bytes per product, which costs 128 x 128 tiles more and the 2 : 1 ones less.  Over 32 shapes
            // from 2560^3 to 16384 x 5120 these numbers' choice is 1.6 % behind the best tile on average and FP8's 4.2 %; they differ on
            // eleven.  The 128 x 128 tiles were slower then; 256 x 128 / 128 x 128 now, microseconds: 4096 x 5120 x 3072 118 / 120, x 4096 152 / 150, 8192 x 1024 x 4096
            // 55 / 60, 16384 x 1280 x 5120 185 / 193; and where they lose, 4096 x 5120 x 2048 84 / 82, 2560^3 40 / 38.  Where a larger tile is far ahead, 4096 x 5120 x 3072 90
            // and 16384 x 1280 x 5120 138 with 256 x 320, better_tile takes it.)
            const double e = per_cu == 2 ? (bf16 ? 0.66 : T <= 3072 ? 0.90 : 0.80) : bf16 && ni * nj == 8 ? 0.80 : eff[ni][nj];
            // a ragged last round may be shared out among all CUs (choose_split): the model's gain scales the cost
            const SplitChoice sc = choose_split((int)tiles, (int)(T / BK), (int)slots, ni, nj, scratch_bytes);
            const double cost = (double)rounds * per_cu * ni * nj / e * (sc.cost_us / sc.whole_cost_us);
            if (best.ni == 0 || cost < best_cost * 0.97) { best = {ni, nj}; best_cost = cost; }   // larger tile on near ties
        }
    return best;
}

// The choice of choose_tile as a plan, and what sharing out its last round of tiles saves.
struct WholePlan {
    TilePlan tile;
    SplitChoice split;
};
static WholePlan plan_whole(int64_t R, int64_t C, int64_t T, int num_cus, bool bf16, size_t scratch_bytes) {
    WholePlan p{{0, 0, kNoEdge}, {}};
    const TileChoice tc = choose_tile(R, C, T, num_cus, scratch_bytes, bf16);
    if (tc.ni == 0) return p;
    p.tile = {tc.ni, tc.nj, kNoEdge};
    p.split = choose_split((int)((R / (64 * tc.ni)) * (C / (64 * tc.nj))), (int)(T / BK), resident_slots(num_cus, tc.ni, tc.nj), tc.ni, tc.nj, scratch_bytes);
    return p;
}

TilePlan plan_tile(int64_t R, int64_t C, int64_t T, int num_cus, bool ta, bool tb, bool slabs_a, bool slabs_b, bool accumulate, bool with_amax, bool bf16,
                   size_t scratch_bytes) {
    WholePlan p = plan_whole(R, C, T, num_cus, bf16, ta || tb || bf16 ? 0 : scratch_bytes);
    if (p.tile.ni) {
        // better_tile prices whole tiles, so a tile of its choice is computed whole, scratch or not: gemm_scratch_bytes has nothing for it (1024 x 24320 x 8192,
        // where 256 x 256 tiles replace smaller ones).
        TilePlan tile = better_tile(R, C, T, num_cus, ta, tb, slabs_a, slabs_b, accumulate, p.tile, p.split.cost_us / p.split.whole_cost_us, p.split.n_groups > 0);
        tile.shares = p.split.n_groups > 0 && tile.ni == p.tile.ni && tile.nj == p.tile.nj && tile.edge == kNoEdge;
        return tile;
    }
    if (!ta || tb) {
        const EdgeChoice ec = choose_edge_tile(R, C, T, num_cus, ta, tb, slabs_a, slabs_b, accumulate, with_amax, bf16);
        p.tile = {ec.ni, ec.nj, ec.edge};
    }
    return better_tile(R, C, T, num_cus, ta, tb, slabs_a, slabs_b, accumulate, p.tile, 1.0);
}

// What a contraction of operands in rows or slabs takes: small tiles of `side`, or (0) the tile; the generic kernel if that has no size either.
struct RowsPlan {
    int side;
    TilePlan tile;
};
static RowsPlan plan_rows(int64_t R, int64_t C, int64_t T, int num_cus, bool slabs_a, bool slabs_b, bool accumulate, bool with_amax, bool bf16, size_t scratch_bytes) {
    // (an operand in slabs is addressed with 32-bit offsets from its first tile row, 0x7FFFFF00 being out of range)
    const int64_t lim = 0x7FFFFF00ll - ((int64_t)1 << 24);
    RowsPlan plan{0, {0, 0, kNoEdge}};
    if ((slabs_a && (T + 256) * R >= lim) || (slabs_b && (T + 256) * C >= lim)) return plan;
    double shared_us = 0.0;
    if (!bf16 && scratch_bytes && T >= 64 * BK && ((R + 127) / 128) * ((C + 127) / 128) <= num_cus) {       // (what the planner shares is that long)
        const WholePlan p = plan_whole(R, C, T, num_cus, false, scratch_bytes);
        if (p.tile.ni) shared_us = shared_tiles_us(p.split);
    }
    plan.side = takes_mini(R, C, T, slabs_a, slabs_b, accumulate, with_amax, bf16, num_cus, shared_us);
    if (plan.side == 0) plan.tile = plan_tile(R, C, T, num_cus, false, false, slabs_a, slabs_b, accumulate, with_amax, bf16, scratch_bytes);
    return plan;
}

template <int FA, int FB>
static void launch_mini(int side, const uint8_t* A, const uint8_t* B, int64_t R, int64_t C, int64_t T, const float* sA, const float* sB,
                        void* c, int accumulate, unsigned* amax, hipStream_t stream, bool slabs_a, bool slabs_b) {
    const int tiles_r = (int)((R + side - 1) / side), tiles = tiles_r * (int)((C + side - 1) / side), grid = (tiles + kXcds - 1) / kXcds * kXcds;
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(kGemmThreads), 0, stream, A, B, reinterpret_cast<uint16_t*>(c), (int)R, (int)C, (int)T, sA, sB, accumulate, amax,
                           slabs_a ? BK : (int)T, slabs_b ? BK : (int)T, slabs_a ? (int)(R * BK) : BK, slabs_b ? (int)(C * BK) : BK, tiles_r, tiles);
    };
    if (side == 32) launch(gemm_mini_kernel<FA, FB, 32>);
    else launch(gemm_mini_kernel<FA, FB, 64>);
}

template <int FA, int FB>
static void launch_one(const uint8_t* A, const uint8_t* B, int64_t R, int64_t C, int64_t T,
                       const float* sA, const float* sB, void* c, int accumulate, unsigned* amax,
                       hipStream_t stream, int num_cus, GemmScratch scratch, bool slabs_a = false, bool slabs_b = false) {
    const RowsPlan plan = plan_rows(R, C, T, num_cus, slabs_a, slabs_b, accumulate != 0, amax != nullptr, FA == kFmtBf16, scratch.ptr ? scratch.bytes : 0);
    const TilePlan tile = plan.tile;
    if (plan.side) { launch_mini<FA, FB>(plan.side, A, B, R, C, T, sA, sB, c, accumulate, amax, stream, slabs_a, slabs_b); return; }
    if (tile.ni && tile.edge == kNoEdge && launch_chosen_tile<FA, FB, false, false>(A, B, R, C, T, sA, sB, c, accumulate, amax, stream, num_cus, tile.shares ? scratch : GemmScratch{}, slabs_a, slabs_b, tile)) return;
    if (tile.ni && launch_edge_tile<FA, FB, false, false>(A, B, R, C, T, sA, sB, c, accumulate, amax, stream, num_cus, slabs_a, slabs_b, tile)) return;
    if constexpr (FA == kFmtBf16) {
        const int64_t n = R * C;
        int64_t blocks = (n + 255) / 256;
        if (blocks > 65536) blocks = 65536;
        hipLaunchKernelGGL(gemm_bf16_generic_kernel, dim3((unsigned)blocks), dim3(256), 0, stream,
                           reinterpret_cast<const uint16_t*>(A), reinterpret_cast<const uint16_t*>(B),
                           reinterpret_cast<uint16_t*>(c), R, C, T / 2, accumulate);
    } else {
        launch_gemm_generic(A, FA, slabs_a ? kLayoutSlabs : kLayoutRows, B, FB, slabs_b ? kLayoutSlabs : kLayoutRows, R, C, T, sA, sB, c,
                            accumulate, amax, stream);
    }
}

void launch_gemm_generic(const uint8_t* A, int fmtA, int ta, const uint8_t* B, int fmtB, int tb, int64_t R, int64_t C,
                         int64_t T, const float* sA, const float* sB, void* c, int accumulate, unsigned* amax,
                         hipStream_t stream) {
    dim3 grid((unsigned)((C + 31) / 32), (unsigned)((R + 31) / 32));
    uint16_t* out = reinterpret_cast<uint16_t*>(c);
    if (fmtA == 0 && fmtB == 0) hipLaunchKernelGGL((gemm_generic_kernel<0, 0>), grid, dim3(256), 0, stream, A, B, out, R, C, T, sA, sB, accumulate, amax, (int)ta, (int)tb);
    else if (fmtA == 1 && fmtB == 0) hipLaunchKernelGGL((gemm_generic_kernel<1, 0>), grid, dim3(256), 0, stream, A, B, out, R, C, T, sA, sB, accumulate, amax, (int)ta, (int)tb);
    else if (fmtA == 0 && fmtB == 1) hipLaunchKernelGGL((gemm_generic_kernel<0, 1>), grid, dim3(256), 0, stream, A, B, out, R, C, T, sA, sB, accumulate, amax, (int)ta, (int)tb);
    else hipLaunchKernelGGL((gemm_generic_kernel<1, 1>), grid, dim3(256), 0, stream, A, B, out, R, C, T, sA, sB, accumulate, amax, (int)ta, (int)tb);
}

void launch_gemm_amax_reset(unsigned* amax, hipStream_t stream) {
    hipLaunchKernelGGL(gemm_amax_reset_kernel, dim3(1), dim3(64), 0, stream, amax);
}

int launch_gemm_tn(const uint8_t* A, int fmtA, const uint8_t* B, int fmtB, int64_t R, int64_t C,
                   int64_t T, const float* d_scaleA, const float* d_scaleB, void* c_bf16,
                   int accumulate, float* d_amax_c, bool amax_is_zeroed, hipStream_t stream, int num_cus, GemmScratch scratch,
                   bool slabs_a, bool slabs_b) {
    unsigned* amax = reinterpret_cast<unsigned*>(d_amax_c);
    if (amax && !amax_is_zeroed) hipLaunchKernelGGL(gemm_amax_reset_kernel, dim3(1), dim3(64), 0, stream, amax);
    if (fmtA == 0 && fmtB == 0) launch_one<0, 0>(A, B, R, C, T, d_scaleA, d_scaleB, c_bf16, accumulate, amax, stream, num_cus, scratch, slabs_a, slabs_b);
    else if (fmtA == 1 && fmtB == 0) launch_one<1, 0>(A, B, R, C, T, d_scaleA, d_scaleB, c_bf16, accumulate, amax, stream, num_cus, scratch, slabs_a, slabs_b);
    else if (fmtA == 0 && fmtB == 1) launch_one<0, 1>(A, B, R, C, T, d_scaleA, d_scaleB, c_bf16, accumulate, amax, stream, num_cus, scratch, slabs_a, slabs_b);
    else launch_one<1, 1>(A, B, R, C, T, d_scaleA, d_scaleB, c_bf16, accumulate, amax, stream, num_cus, scratch, slabs_a, slabs_b);
    return hipGetLastError() == hipSuccess ? 0 : -6;
}

// Scratch a launch of this shape would use when given as much as it likes, with or without addition to the output and its absmax (0: every tile is
// computed whole).
size_t gemm_scratch_bytes(int64_t R, int64_t C, int64_t T, int num_cus) {
    const size_t unlimited = ~(size_t)0;
    const WholePlan p = plan_whole(R, C, T, num_cus, false, unlimited);
    if (p.tile.ni == 0 || p.split.n_groups == 0) return 0;
    const size_t bytes = p.split.slots * (size_t)(4 * 4096 * p.tile.ni * p.tile.nj);
    // shared out unless another kernel takes the shape: small tiles, whole larger ones (plan_tile: the same with addition and without)
    for (int with = 0; with < 4; ++with) {
        const RowsPlan plan = plan_rows(R, C, T, num_cus, false, false, (with & 1) != 0, (with & 2) != 0, false, unlimited);
        if (plan.side == 0) return plan.tile.shares ? bytes : 0;
    }
    return 0;
}

// Phase stamps of the 256 x 256 tile kernel (E4M3 x E4M3, contraction-contiguous operands): the same kernel with
// kProfile, which makes wave 0 of every workgroup record cycle and 100 MHz stamps of its phases, 16 words of 64 bits
// per workgroup id (see GemmTuning::kProfile).
template <bool IEEE>
struct GemmPhaseTuning : GemmTuning {
    static constexpr bool kProfile = true;
    static constexpr bool kIeeeMaximum = IEEE;
    static __device__ void record(float* buf, int block, int slot, long long value) {
        reinterpret_cast<long long*>(buf)[(size_t)block * 16 + slot] = value;
    }
};

int gemm_phase_stamp_blocks(int64_t R, int64_t C) { return (int)((((R / 256) * (C / 256) + kXcds - 1) / kXcds) * kXcds); }

int launch_gemm_phase_stamps(const uint8_t* A, const uint8_t* B, int64_t R, int64_t C, int64_t T, const float* sA,
                             const float* sB, void* c_bf16, float* d_amax_c, long long* stamps, int ieee_maximum,
                             hipStream_t stream, int num_cus) {
    const int tiles_r = (int)(R / 256), tiles_c = (int)(C / 256), nt = tiles_r * tiles_c;
    const int grid = gemm_phase_stamp_blocks(R, C);
    const int slots = resident_slots(num_cus, 4, 4);
    const int band = band_rows();
    const int share_b = band < tiles_r ? band : tiles_r, share_a = 4 < tiles_c ? 4 : tiles_c;
    const int next_stride = successor_stride(4, 4, nt, slots);
    SplitPlan plan{};
    plan.n_whole = nt;
    plan.partials = reinterpret_cast<float*>(stamps);
    unsigned* amax = reinterpret_cast<unsigned*>(d_amax_c);
    hipLaunchKernelGGL(gemm_amax_reset_kernel, dim3(1), dim3(64), 0, stream, amax);
    auto launch = [&](auto kernel) {
        hipLaunchKernelGGL(kernel, dim3(grid), dim3(kGemmThreads), 0, stream, A, B, reinterpret_cast<uint16_t*>(c_bf16),
                           (int)C, (int)T, sA, sB, amax, tiles_r, tiles_c, touch_ahead(), band, next_stride, (int)T, (int)T,
                           BK, BK, share_a, share_b, plan, (int)R, 0);
    };
    if (ieee_maximum) launch(gemm_tile_kernel<0, 0, 4, 4, false, GemmPhaseTuning<true>>);
    else launch(gemm_tile_kernel<0, 0, 4, 4, false, GemmPhaseTuning<false>>);
    return hipGetLastError() == hipSuccess ? 0 : -6;
}

// BF16 baseline: same tile kernels with the BF16 MFMA; T counts elements here, rows are 2 T bytes long.
int launch_gemm_bf16_tn(const void* A, const void* B, int64_t R, int64_t C, int64_t T, void* c_bf16,
                        int accumulate, hipStream_t stream, int num_cus) {
    launch_one<kFmtBf16, kFmtBf16>(reinterpret_cast<const uint8_t*>(A), reinterpret_cast<const uint8_t*>(B), R, C, 2 * T,
                                   nullptr, nullptr, c_bf16, accumulate, nullptr, stream, num_cus, GemmScratch{nullptr, 0});
    return hipGetLastError() == hipSuccess ? 0 : -6;
}

}  // namespace llmq
