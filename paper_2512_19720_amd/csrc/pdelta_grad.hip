// Gradient of a loss with respect to the scale vector v, given dY = dL/dY (paper, algorithm
// "Train per-row/column scaling vectors via activation matching": the loss is backpropagated
// through v only).  With Y[m,o] = sum_i X[m,i] (W_b[o,i] + v. B[o,i])  (Eq. 1 in the layer):
//   row:  dL/dv[o] = sum_m dY[m,o] * (X B^T)[m,o]
//   col:  dL/dv[i] = sum_m X[m,i]  * (dY B)[m,i]
// Both are one matrix product with the +-1 matrix followed by an elementwise product and a sum
// over the tokens; W_b is not needed.  Column mode is row mode with the roles of X and dY
// swapped and the sign matrix transposed, so the library transposes the packed bits once into
// the workspace and runs the same kernel.
//
// Kernel: the prefill tile (256 tokens x 128 outputs x 64 inputs, 8 waves of 64 x 64, MFMA
// 32x32x16 in the operands' own dtype: +-1 is exact in fp16 and bf16, so nothing is converted).
// The epilogue multiplies each accumulator by its G entry and sums the tile's 256 tokens; tiles
// write one partial per (token tile, output) to the workspace and a second kernel adds the
// partials in a fixed order: no atomics, reproducible.
#include <algorithm>
#include <type_traits>

#include "pdelta.h"
#include "pdelta_device.h"
#include "pdelta_host.h"
#include "pdelta_lds_load.h"

namespace pdelta {

constexpr int kGradBM = 256, kGradBN = 128, kGradBK = 64;
constexpr int kGradLDK = kGradBK + 8;                 // LDS row in halves (144 bytes)

template <int DT>
__device__ __forceinline__ float16v grad_mfma(uint4v a, uint4v b, float16v c) {
    if constexpr (DT == kBF16)
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                                       __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(half8, a),
                                                      __builtin_bit_cast(half8, b), c, 0, 0, 0);
}

// Eight sign bits (bit e <-> element e, 1 = +1) to eight +-1.0 values of dtype DT.
template <int DT>
__device__ __forceinline__ uint4v grad_expand(uint32_t byte) {
    constexpr uint32_t one2 = DT == kBF16 ? 0x3F803F80u : 0x3C003C00u;
    const uint32_t neg = ~byte & 0xFFu;               // higher bits would leak into bit 31 below
    uint4v r;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const uint32_t spread = (neg << (30 - 2 * p)) | (neg << (15 - 2 * p));
        r[p] = (spread & 0x80008000u) | one2;
    }
    return r;
}

// partial[tile_m][n] = sum over the tile's tokens m of G[m,n] * sum_k A[m,k] S[n,k],
// A [M, Kc], G [M, Nc], S = +-1 from bits [Nc][Kc/32]; Kc % 32 == 0.
template <int DT>
__global__ void __launch_bounds__(512, 4)
grad_tile_kernel(const uint16_t* __restrict__ A, const uint16_t* __restrict__ G,
                 const uint32_t* __restrict__ bits, float* __restrict__ partial, int M, int Nc, int Kc,
                 int m_tiles)
{
    constexpr int BM = kGradBM, BN = kGradBN, BK = kGradBK, LDK = kGradLDK, ROWS = 64, XQ = 4, WQ = 2;
    __shared__ __attribute__((aligned(16))) uint16_t As[BM * LDK];
    __shared__ __attribute__((aligned(16))) uint16_t Ss[BN * LDK];

    const int tile_m = blockIdx.x % m_tiles, tile_n = blockIdx.x / m_tiles;
    const int m0 = tile_m * BM, n0 = tile_n * BN;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;

    // staging role: 8 inputs (16 bytes of A, one sign byte) at column ld_c of rows ld_row + 64 q;
    // rows past the end are clamped (they only feed results that are never used)
    const int ld_row = tid >> 3, ld_c = (tid & 7) * 8;
    const char* abase = (const char*)(A + (int64_t)m0 * Kc);
    const char* sbase = (const char*)bits + (((int64_t)n0 * Kc) >> 3);
    uint32_t aoff[XQ], soff[WQ];
#pragma unroll
    for (int q = 0; q < XQ; ++q) {
        const int row = min(m0 + ld_row + ROWS * q, M - 1) - m0;
        aoff[q] = ((uint32_t)row * (uint32_t)Kc + (uint32_t)ld_c) * 2u;
    }
#pragma unroll
    for (int q = 0; q < WQ; ++q) {
        const int row = min(n0 + ld_row + ROWS * q, Nc - 1) - n0;
        soff[q] = (uint32_t)row * (uint32_t)(Kc >> 3) + (uint32_t)(tid & 7);
    }
    uint4v ag[XQ];
    uint32_t sb[WQ];
    const uint4v zero = {0, 0, 0, 0};
    auto load_global = [&](int kb, auto guard) {
        constexpr bool GUARD = decltype(guard)::value;
        const bool col_ok = !GUARD || kb + ld_c < Kc;
        const char* ab = abase + (int64_t)kb * 2;
        const char* sp = sbase + (kb >> 3);
#pragma unroll
        for (int q = 0; q < XQ; ++q) ag[q] = col_ok ? *(const uint4v*)(ab + aoff[q]) : zero;
#pragma unroll
        for (int q = 0; q < WQ; ++q) sb[q] = col_ok ? (uint32_t) * (const uint8_t*)(sp + soff[q]) : 0xFFu;
    };
    auto store_lds = [&]() {
#pragma unroll
        for (int q = 0; q < XQ; ++q) *(uint4v*)(As + (ld_row + ROWS * q) * LDK + ld_c) = ag[q];
#pragma unroll
        for (int q = 0; q < WQ; ++q) *(uint4v*)(Ss + (ld_row + ROWS * q) * LDK + ld_c) = grad_expand<DT>(sb[q]);
    };

    float16v acc[2][2];
#pragma unroll
    for (int f = 0; f < 2; ++f)
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[f][h][r] = 0.f;

    const int frag_row = lane & 31, frag_k = (lane >> 5) * 8;
    const uint16_t* a_base = As + (wm * 64 + frag_row) * LDK + frag_k;
    const uint16_t* b_base = Ss + (wn * 64 + frag_row) * LDK + frag_k;
    auto multiply_stage = [&]() {
#pragma unroll
        for (int ks = 0; ks < BK / 16; ++ks) {
            uint4v a[2], b[2];
#pragma unroll
            for (int f = 0; f < 2; ++f) a[f] = *(const uint4v*)(a_base + f * 32 * LDK + ks * 16);
#pragma unroll
            for (int h = 0; h < 2; ++h) b[h] = *(const uint4v*)(b_base + h * 32 * LDK + ks * 16);
#pragma unroll
            for (int f = 0; f < 2; ++f)
#pragma unroll
                for (int h = 0; h < 2; ++h) acc[f][h] = grad_mfma<DT>(a[f], b[h], acc[f][h]);
        }
    };

    const int full_steps = Kc / BK;
    const bool tail = (Kc % BK) != 0;                 // then one more step of 32 inputs
    if (full_steps > 0) load_global(0, std::false_type{});
    else load_global(0, std::true_type{});
    for (int i = 0; i + 1 < full_steps; ++i) {
        store_lds();
        __syncthreads();
        load_global((i + 1) * BK, std::false_type{});
        __builtin_amdgcn_sched_barrier(0);            // keep the loads above the multiplication
        multiply_stage();
        __syncthreads();
    }
    if (full_steps > 0) {
        store_lds();
        __syncthreads();
        if (tail) load_global(full_steps * BK, std::true_type{});
        multiply_stage();
        __syncthreads();
    }
    if (tail) {
        store_lds();
        __syncthreads();
        multiply_stage();
        __syncthreads();
    }

    // epilogue: acc[f][h][r] is token m0 + 64 wm + 32 f + 8 (r / 4) + 4 (lane / 32) + r % 4,
    // output n0 + 64 wn + 32 h + lane % 32.  Multiply by G, sum the wave's 64 tokens, then the
    // four token groups of the tile in LDS (As is free now).
    float* red = (float*)As;                           // [4 wm][128]
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int n = n0 + wn * 64 + h * 32 + (lane & 31);
        const int nc = min(n, Nc - 1);
        float s = 0.f;
#pragma unroll
        for (int f = 0; f < 2; ++f)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int tok = m0 + wm * 64 + f * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
                const uint32_t gbits = G[(int64_t)min(tok, M - 1) * Nc + nc];
                const float gval = tok < M ? bits_to_f32<DT>(gbits) : 0.f;
                s += gval * acc[f][h][r];
            }
        s += __shfl_xor(s, 32, kWave);
        if (lane < 32) red[wm * BN + wn * 64 + h * 32 + lane] = s;
    }
    __syncthreads();
    if (tid < BN) {
        const int n = n0 + tid;
        if (n < Nc) partial[(int64_t)tile_m * Nc + n] = (red[tid] + red[BN + tid]) + (red[2 * BN + tid] + red[3 * BN + tid]);
    }
}

// Pipelined form of grad_tile_kernel, organised like the prefill kernel of the same tile: one
// workgroup per CU, two LDS stages and two register sets.  During step s a wave multiplies stage
// s % 2 and, between its groups of four MFMAs, stages the operands of step s+1 (loaded one step
// earlier) into the other stage while the loads of step s+2 are in flight: one barrier per step.
struct GradRegs {
    uint4v ag[4];
    uint32_t sb[2];
};

template <int DT>
__global__ void __launch_bounds__(512, 2)
grad_tile_pipe_kernel(const uint16_t* __restrict__ A, const uint16_t* __restrict__ G,
                      const uint32_t* __restrict__ bits, float* __restrict__ partial, int M, int Nc, int Kc,
                      int m_tiles)
{
    constexpr int BM = kGradBM, BN = kGradBN, BK = kGradBK, LDK = kGradLDK, ROWS = 64, XQ = 4, WQ = 2;
    constexpr int AS = BM * LDK, STAGE = (BM + BN) * LDK;                 // halves
    extern __shared__ __attribute__((aligned(16))) unsigned char grad_smem[];
    uint16_t* lds = (uint16_t*)grad_smem;                                 // [2][STAGE]: A tile then sign tile

    const int tile_m = blockIdx.x % m_tiles, tile_n = blockIdx.x / m_tiles;
    const int m0 = tile_m * BM, n0 = tile_n * BN;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;

    const int ld_row = tid >> 3, ld_c = (tid & 7) * 8;
    const char* abase = (const char*)(A + (int64_t)m0 * Kc);
    const char* sbase = (const char*)bits + (((int64_t)n0 * Kc) >> 3);
    uint32_t aoff[XQ], soff[WQ];
#pragma unroll
    for (int q = 0; q < XQ; ++q) {
        const int row = min(m0 + ld_row + ROWS * q, M - 1) - m0;
        aoff[q] = ((uint32_t)row * (uint32_t)Kc + (uint32_t)ld_c) * 2u;
    }
#pragma unroll
    for (int q = 0; q < WQ; ++q) {
        const int row = min(n0 + ld_row + ROWS * q, Nc - 1) - n0;
        soff[q] = (uint32_t)row * (uint32_t)(Kc >> 3) + (uint32_t)(tid & 7);
    }
    const uint4v zero = {0, 0, 0, 0};
    auto load_global = [&](GradRegs& R, int kb, auto guard) {
        constexpr bool GUARD = decltype(guard)::value;
        const bool col_ok = !GUARD || kb + ld_c < Kc;
        const char* ab = abase + (int64_t)kb * 2;
        const char* sp = sbase + (kb >> 3);
#pragma unroll
        for (int q = 0; q < XQ; ++q) R.ag[q] = col_ok ? *(const uint4v*)(ab + aoff[q]) : zero;
#pragma unroll
        for (int q = 0; q < WQ; ++q) R.sb[q] = col_ok ? (uint32_t) * (const uint8_t*)(sp + soff[q]) : 0xFFu;
    };
    // quarter c of the staging work of one step
    auto stage_part = [&](const GradRegs& R, uint16_t* stage, int c) {
        if (c < 2) {
            *(uint4v*)(stage + AS + (ld_row + ROWS * c) * LDK + ld_c) = grad_expand<DT>(R.sb[c]);
            *(uint4v*)(stage + (ld_row + ROWS * c) * LDK + ld_c) = R.ag[c];
        } else {
            *(uint4v*)(stage + (ld_row + ROWS * c) * LDK + ld_c) = R.ag[c];
        }
    };

    float16v acc[2][2];
#pragma unroll
    for (int f = 0; f < 2; ++f)
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[f][h][r] = 0.f;

    const int frag_row = lane & 31, frag_k = (lane >> 5) * 8;
    const int a_off = (wm * 64 + frag_row) * LDK + frag_k;
    const int b_off = AS + (wn * 64 + frag_row) * LDK + frag_k;
    auto step = [&](const uint16_t* rd, uint16_t* wr, const GradRegs& Rnext, bool stage_next) {
        uint4v a[2][2], b[2][2];
#pragma unroll
        for (int f = 0; f < 2; ++f) a[0][f] = *(const uint4v*)(rd + a_off + f * 32 * LDK);
#pragma unroll
        for (int h = 0; h < 2; ++h) b[0][h] = *(const uint4v*)(rd + b_off + h * 32 * LDK);
#pragma unroll
        for (int ks = 0; ks < BK / 16; ++ks) {
            const int cur = ks & 1, nxt = cur ^ 1;
#pragma unroll
            for (int f = 0; f < 2; ++f)
#pragma unroll
                for (int h = 0; h < 2; ++h) acc[f][h] = grad_mfma<DT>(a[cur][f], b[cur][h], acc[f][h]);
            if (ks + 1 < BK / 16) {
#pragma unroll
                for (int f = 0; f < 2; ++f) a[nxt][f] = *(const uint4v*)(rd + a_off + f * 32 * LDK + (ks + 1) * 16);
#pragma unroll
                for (int h = 0; h < 2; ++h) b[nxt][h] = *(const uint4v*)(rd + b_off + h * 32 * LDK + (ks + 1) * 16);
            }
            if (stage_next) stage_part(Rnext, wr, ks);
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    const int full_steps = Kc / BK;
    const int n_steps = full_steps + ((Kc % BK) != 0 ? 1 : 0);
    auto load_any = [&](GradRegs& R, int s) {
        if (s < full_steps) load_global(R, s * BK, std::false_type{});
        else load_global(R, s * BK, std::true_type{});
    };
    uint16_t* st0 = lds;
    uint16_t* st1 = lds + STAGE;
    GradRegs R0, R1;
    load_any(R0, 0);
    if (n_steps > 1) load_any(R1, 1);
#pragma unroll
    for (int c = 0; c < 4; ++c) stage_part(R0, st0, c);
    __syncthreads();

    int s = 0;
    // steady state, two steps per iteration (stages and register sets static); the loads are
    // unconditional and unguarded, so that their waits stay as deep as the pipeline
    for (; s + 3 < full_steps; s += 2) {
        load_global(R0, (s + 2) * BK, std::false_type{});
        __builtin_amdgcn_sched_barrier(0);
        step(st0, st1, R1, true);
        __syncthreads();
        load_global(R1, (s + 3) * BK, std::false_type{});
        __builtin_amdgcn_sched_barrier(0);
        step(st1, st0, R0, true);
        __syncthreads();
    }
    // the last (up to three, possibly one partial) steps
    for (; s < n_steps; ++s) {
        const bool even = (s & 1) == 0;
        if (s + 2 < n_steps) {
            if (even) load_any(R0, s + 2); else load_any(R1, s + 2);
        }
        const bool more = s + 1 < n_steps;
        if (even) step(st0, st1, R1, more); else step(st1, st0, R0, more);
        __syncthreads();
    }

    // epilogue as in grad_tile_kernel (every step ended with a barrier: the stages are free)
    float* red = (float*)lds;                          // [4 wm][128]
#pragma unroll
    for (int h = 0; h < 2; ++h) {
        const int n = n0 + wn * 64 + h * 32 + (lane & 31);
        const int nc = min(n, Nc - 1);
        float sum = 0.f;
#pragma unroll
        for (int f = 0; f < 2; ++f)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int tok = m0 + wm * 64 + f * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
                const uint32_t gbits = G[(int64_t)min(tok, M - 1) * Nc + nc];
                const float gval = tok < M ? bits_to_f32<DT>(gbits) : 0.f;
                sum += gval * acc[f][h][r];
            }
        sum += __shfl_xor(sum, 32, kWave);
        if (lane < 32) red[wm * BN + wn * 64 + h * 32 + lane] = sum;
    }
    __syncthreads();
    if (tid < BN) {
        const int n = n0 + tid;
        if (n < Nc) partial[(int64_t)tile_m * Nc + n] = (red[tid] + red[BN + tid]) + (red[2 * BN + tid] + red[3 * BN + tid]);
    }
}

template <int DT>
static int launch_grad_tile_pipe(const uint16_t* A, const uint16_t* G, const uint32_t* bits, float* partial,
                                 int M, int Nc, int Kc, int m_tiles, unsigned grid, hipStream_t stream)
{
    constexpr size_t lds = (size_t)2 * (kGradBM + kGradBN) * kGradLDK * sizeof(uint16_t);   // 110,592 bytes
    auto kernel = grad_tile_pipe_kernel<DT>;
    static unsigned lds_opted_in = 0;                 // per template instance: one kernel
    if (opt_in_dynamic_lds((const void*)kernel, (int)lds, &lds_opted_in) != 0) return -1;
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(512), lds, stream, A, G, bits, partial, M, Nc, Kc, m_tiles);
    return 0;
}

// ---------------------------------------------------------------------------------------------
// 256 tokens x 256 outputs x 64 inputs, the form of the 256 x 256 prefill kernel (Kc a multiple of 128):
// A comes by direct loads into LDS, the sign tile is expanded from sign words that were fetched for four
// steps at a time, two LDS stages, one barrier per step three quarters into it.  Half the A traffic per
// product of the 256 x 128 kernel, and none of it through registers.  The contraction may be cut into
// `parts`, each with partial sums of its own: the epilogue is linear, so a part costs one more row of
// partials and nothing else.  2048 tokens, 4096 x 4096 bf16: see grad_big_parts.
constexpr int kGbTile = 256, kGbBK = 64, kGbUnitK = 128;
constexpr int kGbAB = kGbTile * kGbBK * 2, kGbStage = 2 * kGbAB;      // bytes of A (of the signs) and of a stage
// behind the stages, per wave: sign words (1 KB), and where touched lines of G end up (256 B)
constexpr int kGbSigns = 2 * kGbStage, kGbTouch = kGbSigns + 8 * 1024, kGbLds = kGbTouch + 8 * 256;

template <int DT>
__global__ void __launch_bounds__(512, 2)
grad_big_kernel(const uint16_t* __restrict__ A, const uint16_t* __restrict__ G, const uint32_t* __restrict__ bits,
                float* __restrict__ partial, int M, int Nc, int Kc, int m_tiles, int tiles, int parts)
{
    constexpr int FM = 4, FN = 2;                     // a wave owns 128 tokens x 64 outputs
    extern __shared__ __attribute__((aligned(16))) unsigned char gb_smem[];

    // each XCD takes a contiguous range of units: token tiles first, then output tiles, then parts
    const int units = tiles * parts, per = (units + 7) / 8;
    const int unit = (int)(blockIdx.x % 8) * per + (int)blockIdx.x / 8;
    if (unit >= units) return;                        // whole workgroup
    const int part = unit / tiles, tile = unit % tiles;
    const int tile_m = tile % m_tiles, m0 = tile_m * kGbTile, n0 = tile / m_tiles * kGbTile;
    const int k_units = Kc / kGbUnitK;
    const int k_first = (int)((int64_t)k_units * part / parts), k_end = (int)((int64_t)k_units * (part + 1) / parts);
    const int n_steps = (k_end - k_first) * (kGbUnitK / kGbBK);       // even, at least 2
    const int kb0 = k_first * kGbUnitK, kb_end = k_end * kGbUnitK;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int wm = wave >> 2, wn = wave & 3;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)gb_smem;

    // A load covers 8 rows of 128 bytes, a wave loads 32 rows of A and expands 32 rows of signs; rows past
    // the end repeat the last one (they only feed results that are never used).  The 16-byte piece p of LDS
    // row r holds inputs 8 (p ^ ((r >> 1) & 7)) .. +7.
    const char* abase = (const char*)(A + (int64_t)m0 * Kc + kb0);
    uint32_t chunk[2], aoff[4];
#pragma unroll
    for (int q = 0; q < 2; ++q) chunk[q] = (uint32_t)((lane & 7) ^ (q * 4 + (lane >> 4)));
#pragma unroll
    for (int q = 0; q < 4; ++q)
        aoff[q] = (uint32_t)(min(m0 + wave * 32 + q * 8 + (lane >> 3), M - 1) - m0) * (uint32_t)Kc * 2u + chunk[q & 1] * 16u;
    // lanes 0-31: sign words of the wave's rows for two steps, lanes 32-63 for the next two
    const int srow = min(n0 + wave * 32 + (lane & 31), Nc - 1);
    const char* sptr = (const char*)bits + (int64_t)srow * (Kc >> 3) + (kb0 >> 3);

    auto request = [&](int s, uint32_t stage) {
        const int rel = s * kGbBK;
        if ((s & 3) == 0) {                           // never past Kc: a short last group repeats its first half
            const int half = (lane >= 32 && kb0 + rel + 128 < kb_end) ? 16 : 0;
            load_lds_16v(lds0 + kGbSigns + wave * 1024, sptr + (rel >> 3) + half);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) load_lds_16(lds0 + stage + (wave * 4 + q) * 1024, aoff[q], abase + (int64_t)rel * 2);
    };
    uint32_t sbyte[4];
    auto fetch_signs = [&](int s) {
        const unsigned char* signs = gb_smem + kGbSigns + wave * 1024 + ((s >> 1) & 1) * 512 + (s & 1) * 8;
#pragma unroll
        for (int q = 0; q < 4; ++q) sbyte[q] = signs[(q * 8 + (lane >> 3)) * 16 + chunk[q & 1]];
    };
    auto expand = [&](uint32_t stage) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint32_t neg = ~sbyte[q] & 0xFFu;
            uint32_t y = neg | (neg << 15);           // bit 2p + 1 at 2p + 16
            asm("" : "+v"(y));                        // (else y and its shifts become full multiplications)
            uint4v r;
#pragma unroll
            for (int p = 0; p < 4; ++p) r[p] = ((y << (15 - 2 * p)) & 0x80008000u) | (DT == kBF16 ? 0x3F803F80u : 0x3C003C00u);
            *(uint4v*)(gb_smem + stage + kGbAB + (wave * 4 + q) * 1024 + lane * 16) = r;
        }
    };

    float16v acc[FM][FN];
#pragma unroll
    for (int f = 0; f < FM; ++f)
#pragma unroll
        for (int h = 0; h < FN; ++h)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[f][h][r] = 0.f;

    uint32_t frag[4];                                 // byte offset of this lane's piece of 16 inputs ks
#pragma unroll
    for (int ks = 0; ks < 4; ++ks)
        frag[ks] = (uint32_t)((lane & 31) * 128 + (((ks * 2 + (lane >> 5)) ^ ((lane >> 1) & 7)) * 16));
    uint4v a[2][FM], b[2][FN];
    auto read_frags = [&](uint32_t stage, int ks) {
        const unsigned char* xa = gb_smem + stage + wm * 128 * 128 + frag[ks];
        const unsigned char* sa = gb_smem + stage + kGbAB + wn * 64 * 128 + frag[ks];
#pragma unroll
        for (int h = 0; h < FN; ++h) b[ks & 1][h] = *(const uint4v*)(sa + h * 32 * 128);
#pragma unroll
        for (int f = 0; f < FM; ++f) a[ks & 1][f] = *(const uint4v*)(xa + f * 32 * 128);
    };
    auto multiply = [&](int ks) {
#pragma unroll
        for (int f = 0; f < FM; ++f)
#pragma unroll
            for (int h = 0; h < FN; ++h) acc[f][h] = grad_mfma<DT>(a[ks & 1][f], b[ks & 1][h], acc[f][h]);
    };

    request(0, 0);
    wait_loads<0>();
    fetch_signs(0);
    expand(0);
    lds_barrier();
    request(1, kGbStage);
    read_frags(0, 0);

    // The tile's lines of G, on their way to L2 during the last two steps (two 128-byte lines per thread; the data goes
    // to LDS that nobody reads): the epilogue would wait for memory eight times otherwise.
    const char* gbase = (const char*)(G + (int64_t)m0 * Nc);
    auto touch_g = [&]() {
        const uint32_t row = (uint32_t)(min(m0 + (int)threadIdx.x / 2, M - 1) - m0) * (uint32_t)Nc;
#pragma unroll
        for (int q = 0; q < 2; ++q)
            load_lds_2(lds0 + kGbTouch + wave * 256, (row + (uint32_t)min(n0 + ((int)threadIdx.x % 2 * 2 + q) * 64, Nc - 1)) * 2u, gbase);
    };

    // Step s; REQ: request step s + 2, MORE: there is a step s + 1.  The fences keep the LDS reads above
    // the MFMAs and the expansion between them.
    auto step = [&](int s, uint32_t cur, uint32_t nxt, auto req, auto more) {
        constexpr bool REQ = decltype(req)::value, MORE = decltype(more)::value;
        read_frags(cur, 1);
        __builtin_amdgcn_sched_barrier(0);
        multiply(0);
        __builtin_amdgcn_sched_barrier(0);
        read_frags(cur, 2);
        __builtin_amdgcn_sched_barrier(0);
        multiply(1);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (REQ) wait_loads<0>();
        else if constexpr (MORE) wait_loads<2>();     // (all but touch_g)
        if constexpr (MORE) fetch_signs(s + 1);
        read_frags(cur, 3);
        __builtin_amdgcn_sched_barrier(0);
        multiply(2);
        if constexpr (MORE) { expand(nxt); interleave<FM * FN, 6>(); }
        __builtin_amdgcn_sched_barrier(0);
        lds_barrier();
        if constexpr (MORE) read_frags(nxt, 0);
        if constexpr (REQ) request(s + 2, cur);
        __builtin_amdgcn_sched_barrier(0);
        multiply(3);
        __builtin_amdgcn_sched_barrier(0);
    };
    int s = 0;
    for (; s + 2 < n_steps; s += 2) {
        step(s, 0, kGbStage, std::true_type{}, std::true_type{});
        step(s + 1, kGbStage, 0, std::true_type{}, std::true_type{});
    }
    touch_g();
    step(s, 0, kGbStage, std::false_type{}, std::true_type{});
    step(s + 1, kGbStage, 0, std::false_type{}, std::false_type{});

    // epilogue as in grad_tile_kernel, a sum of its own for each 32 tokens (the last barrier came after the
    // last fragment read: the stages are free).  The 128 entries of G that a lane needs are asked for 16 at a time, one
    // group ahead of the sums, from uniform row addresses; rows past the end repeat the last one and count as zero.
    // Left to itself the compiler puts every 2-byte load behind a branch on its token and waits for it, 20 us a tile.
    float* red = (float*)gb_smem;                      // [2 wm][256]
    const int tok0 = m0 + wm * 128, half4 = (lane >> 5) * 4;
    uint32_t gbits[2][16], goff[FN];
#pragma unroll
    for (int h = 0; h < FN; ++h) goff[h] = (uint32_t)min(n0 + wn * 64 + h * 32 + (lane & 31), Nc - 1) * 2u;
    const uint32_t gstep = (uint32_t)half4 * (uint32_t)Nc * 2u;
    auto weighted_sums = [&](auto full) {
        constexpr bool FULL = decltype(full)::value;  // all of the tile's tokens exist
        auto load_g = [&](int i) {
            const int h = i / FM, f = i % FM;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int row = wm * 128 + f * 32 + (r >> 2) * 8 + (r & 3);
                if constexpr (FULL)
                    gbits[i & 1][r] = *(const uint16_t*)(gbase + (int64_t)row * Nc * 2 + (goff[h] + gstep));
                else
                    gbits[i & 1][r] = *(const uint16_t*)(gbase + ((uint32_t)(min(m0 + row + half4, M - 1) - m0) * (uint32_t)Nc * 2u + goff[h]));
            }
        };
        load_g(0);
        float t = 0.f, first = 0.f;
#pragma unroll
        for (int i = 0; i < FN * FM; ++i) {
            const int h = i / FM, f = i % FM;
            if (i + 1 < FN * FM) load_g(i + 1);
            __builtin_amdgcn_sched_barrier(0);
            float sum = 0.f;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                uint32_t g = gbits[i & 1][r];
                if constexpr (!FULL) g = tok0 + f * 32 + (r >> 2) * 8 + half4 + (r & 3) < M ? g : 0u;
                sum += bits_to_f32<DT>(g) * acc[f][h][r];
            }
            __builtin_amdgcn_sched_barrier(0);
            if ((f & 1) == 0) first = sum;
            else t = f == 1 ? first + sum : t + (first + sum);
            if (f == FM - 1) {
                t += __shfl_xor(t, 32, kWave);
                if (lane < 32) red[wm * kGbTile + wn * 64 + h * 32 + lane] = t;
            }
        }
    };
    if (m0 + kGbTile <= M) weighted_sums(std::true_type{});       // uniform
    else weighted_sums(std::false_type{});
    __syncthreads();
    const int tid = threadIdx.x;
    if (tid < kGbTile && n0 + tid < Nc)
        partial[(int64_t)(part * m_tiles + tile_m) * Nc + n0 + tid] = red[tid] + red[kGbTile + tid];
}

// Parts of the contraction for the 256 x 256 kernel, or 0 for the 256 x 128 kernel, which is taken where the
// contraction is not a multiple of 128, the caller's workspace has no room for the parts, or a few tokens meet one or two
// units (one token, 512 x 256 row 9.5 us and 10.9 here; 64: 13.8 and 10.9) or up to five and so many tiles that two parts
// are the most (one token, 22784 x 384 row 12.1 and 14.1, eight, 21888 x 640 15.9 and 17.1; 1152 inputs 21.6 and 22.0).  A round of up to 256
// workgroups takes 4 us and 1.12 us per step of 64 inputs (1.44 when all CUs multiply and the clock falls); a part more
// is one more row of partial sums for the second launch.  Up to 16 parts for at most 128 workgroups (one token, 8192 x 1024
// col 24.9 us, 33.5 with eight; 2048 x 8192 row 20.8 and 29.4), else up to eight.  Changing
// inputs, bf16 row, the 256 x 128 kernel or the earlier epilogue, then now: 64 tokens, 11008 x 4096 65 -> 29 us; 256 tokens,
// 4096 x 4096 42 -> 20; 1024 66 -> 35; 2048 71 -> 54 (col 77 -> 59); 2048 tokens, 11008 x 4096 210 -> 153; 4000 tokens, 2048 x
// 2048 45 -> 33.  Counters, 2048 tokens, 4096 x 4096 col: matrix cores busy 61 % of the CU's cycles, vector ALUs 21 %, LDS 33 %.
static int grad_big_parts(int64_t M, int64_t Nc, int64_t Kc)
{
    const int forced = tune_value("grad_big", -1);     // 0: never; n > 0: in n parts
    if (Kc % kGbUnitK != 0 || M <= 0 || forced == 0 || (forced < 0 && tune_value("grad_pipe", -1) >= 0)) return 0;
    const int64_t m_tiles = (M + kGbTile - 1) / kGbTile, tiles = m_tiles * ((Nc + kGbTile - 1) / kGbTile), units = Kc / kGbUnitK;
    if (tiles > (1 << 24)) return 0;
    if (forced > 0) return (int)std::min<int64_t>(forced, units);
    if (M <= 16 && (units <= 2 || (units <= 5 && tiles > 256 / 3))) return 0;
    const int64_t most = std::max<int64_t>(8, std::min<int64_t>(16, 128 / tiles));
    double best = 0;
    int parts = 0;
    for (int64_t p = 1; p <= std::min(most, units); ++p) {
        const double t = (double)((tiles * p + 255) / 256) * (4 + 1.12 * 2 * (double)((units + p - 1) / p));
        if (parts == 0 || t < best) { best = t; parts = (int)p; }
    }
    return parts;
}

template <int DT>
static int launch_grad_big(const uint16_t* A, const uint16_t* G, const uint32_t* bits, float* partial, int M, int Nc, int Kc,
                           int m_tiles, int parts, hipStream_t stream)
{
    auto kernel = grad_big_kernel<DT>;
    static unsigned lds_opted_in = 0;                 // per template instance: one kernel
    if (opt_in_dynamic_lds((const void*)kernel, kGbLds, &lds_opted_in) != 0) return -1;
    const int tiles = m_tiles * ((Nc + kGbTile - 1) / kGbTile);
    const unsigned grid = (unsigned)((tiles * parts + 7) / 8 * 8);
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(512), kGbLds, stream, A, G, bits, partial, M, Nc, Kc, m_tiles, tiles, parts);
    return 0;
}

// Sums of the partial rows (up to 16 parts times the token tiles) in fp64: a block takes 64 outputs, its wave w the
// rows w, w + 4, ..., so that every load of a thread is in flight at once and 4096 outputs spread over 64 CUs.
__global__ void __launch_bounds__(256)
grad_reduce_kernel(const float* __restrict__ partial, float* __restrict__ grad, int n, int rows)
{
    __shared__ double part[4][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int i = blockIdx.x * 64 + lane, ic = min(i, n - 1);
    double s = 0.0;
#pragma unroll 8
    for (int t = w; t < rows; t += 4) s += (double)partial[(int64_t)t * n + ic];
    part[w][lane] = s;
    __syncthreads();
    if (w == 0 && i < n) grad[i] = (float)((part[0][lane] + part[1][lane]) + (part[2][lane] + part[3][lane]));
}

// Bt[i][o / 32] bit (o % 32) = B[o][i / 32] bit (i % 32); d_out % 32 == 0.  A wave takes 64 rows
// o and one word column: 32 ballots turn the lanes' words into the 64-bit columns.
__global__ void __launch_bounds__(256)
transpose_bits_kernel(const uint32_t* __restrict__ B, uint32_t* __restrict__ Bt, int d_out, int d_in)
{
    const int lane = threadIdx.x & 63;
    const int wcol = blockIdx.x * 4 + (threadIdx.x >> 6);            // word column of B
    const int wpr = d_in >> 5;
    if (wcol >= wpr) return;                                        // whole wave
    const int o = blockIdx.y * 64 + lane;
    const uint32_t word = o < d_out ? B[(int64_t)o * wpr + wcol] : 0u;
    unsigned long long mine = 0;
#pragma unroll
    for (int b = 0; b < 32; ++b) {
        const unsigned long long m = __ballot((word >> b) & 1u);
        if (lane == b) mine = m;
    }
    if (lane < 32) {
        const int i = wcol * 32 + lane;
        const int wpr_t = d_out >> 5;
        const int w0 = blockIdx.y * 2;
        Bt[(int64_t)i * wpr_t + w0] = (uint32_t)mine;
        if (w0 + 1 < wpr_t) Bt[(int64_t)i * wpr_t + w0 + 1] = (uint32_t)(mine >> 32);
    }
}

// The same for large matrices.  A lane transposes one block of 32 x 32 bits in registers by recursive block transposition
// (H. S. Warren, Hacker's Delight, 7-3: five rounds of masked swaps, 10 instructions for each of its words; ballots took eight times that); the
// lanes of a wave take 64 consecutive words of each row, the four waves 128 rows, whose 16 bytes per row of Bt leave
// through LDS as one store.  4096 x 4096: 5.4 us a launch, 7.1 with ballots and 4-byte loads down the columns.
__global__ void __launch_bounds__(256)
transpose_bits_blocks_kernel(const uint32_t* __restrict__ B, uint32_t* __restrict__ Bt, int d_out, int d_in)
{
    constexpr int COL = 32 * 4 + 4;                   // words per word column: [bit][row block], padded
    __shared__ __attribute__((aligned(16))) uint32_t out[64 * COL];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int wpr = d_in >> 5, wpr_t = d_out >> 5;
    const int wcol0 = blockIdx.x * 64, rblock0 = blockIdx.y * 4;
    const int wcol = min(wcol0 + lane, wpr - 1), rblock = min(rblock0 + w, wpr_t - 1);    // (repeats are not stored)
    const uint32_t* src = B + (int64_t)rblock * 32 * wpr + wcol;
    uint32_t a[32];
#pragma unroll
    for (int r = 0; r < 32; ++r) a[r] = src[(int64_t)r * wpr];
    auto trade = [&](auto width) {                    // rows r and r + J trade the halves of their fields of 2 J bits
        constexpr int J = decltype(width)::value;
        constexpr uint32_t low = J == 16 ? 0x0000FFFFu : J == 8 ? 0x00FF00FFu : J == 4 ? 0x0F0F0F0Fu : J == 2 ? 0x33333333u : 0x55555555u;
#pragma unroll
        for (int r = 0; r < 32; ++r) {
            if (r & J) continue;
            const uint32_t x = a[r], y = a[r + J];
            a[r] = (x & low) | ((y << J) & ~low);
            a[r + J] = ((x >> J) & low) | (y & ~low);
        }
    };
    trade(std::integral_constant<int, 16>{});
    trade(std::integral_constant<int, 8>{});
    trade(std::integral_constant<int, 4>{});
    trade(std::integral_constant<int, 2>{});
    trade(std::integral_constant<int, 1>{});
#pragma unroll
    for (int b = 0; b < 32; ++b) out[lane * COL + b * 4 + w] = a[b];
    __syncthreads();
    const bool whole = rblock0 + 4 <= wpr_t && (wpr_t & 3) == 0;              // 16-byte aligned pieces
    for (int k = threadIdx.x; k < 64 * 32; k += 256) {
        if (wcol0 + (k >> 5) >= wpr) break;
        uint32_t* dst = Bt + ((int64_t)wcol0 * 32 + k) * wpr_t + rblock0;
        const uint32_t* from = out + (k >> 5) * COL + (k & 31) * 4;
        if (whole) *(uint4v*)dst = *(const uint4v*)from;
        else
            for (int q = 0; q < 4 && rblock0 + q < wpr_t; ++q) dst[q] = from[q];
    }
}

static size_t grad_bytes(int64_t M, int64_t d_out, int64_t d_in, int axis, int parts)
{
    const int64_t m_tiles = (M + kGradBM - 1) / kGradBM;
    const int64_t n = axis == 0 ? d_out : d_in;
    size_t bytes = (size_t)(m_tiles > 0 ? m_tiles : 1) * parts * n * sizeof(float);
    bytes = (bytes + 255) & ~(size_t)255;
    if (axis == 1) bytes += (size_t)d_in * (d_out / 8);            // transposed sign bits
    return bytes;
}
size_t grad_v_workspace_bytes(int64_t M, int64_t d_out, int64_t d_in, int axis) { return grad_bytes(M, d_out, d_in, axis, 1); }
size_t grad_v_split_workspace_bytes(int64_t M, int64_t d_out, int64_t d_in, int axis)
{
    return grad_bytes(M, d_out, d_in, axis, std::max(1, grad_big_parts(M, axis == 0 ? d_out : d_in, axis == 0 ? d_in : d_out)));
}

int launch_grad_v(int dtype, int axis, const void* X, const void* dY, const uint32_t* B_packed, float* grad,
                  int64_t M, int64_t d_out, int64_t d_in, void* workspace, size_t workspace_bytes, hipStream_t stream)
{
    const int64_t m_tiles = (M + kGradBM - 1) / kGradBM;
    const int64_t Nc = axis == 0 ? d_out : d_in, Kc = axis == 0 ? d_in : d_out;
    int parts = grad_big_parts(M, Nc, Kc);
    if (parts > 1 && grad_bytes(M, d_out, d_in, axis, parts) > workspace_bytes) parts = 0;
    float* partial = (float*)workspace;
    const uint16_t* A = (const uint16_t*)(axis == 0 ? X : dY);
    const uint16_t* G = (const uint16_t*)(axis == 0 ? dY : X);
    const uint32_t* bits = B_packed;
    if (axis == 1 && m_tiles > 0) {
        size_t off = (size_t)m_tiles * std::max(1, parts) * Nc * sizeof(float);
        off = (off + 255) & ~(size_t)255;
        uint32_t* Bt = (uint32_t*)((char*)workspace + off);
        // Above 2^23 signs by blocks in registers, whose few waves each take longer (col gradient of 256 tokens, ballots /
        // blocks: 1024 x 1024 13.9 / 15.0 us, 2048 x 4096 18.7 / 18.9, 4096 x 4096 25.7 / 24.7, 4096 x 11008 41.5 / 34.6).
        // Rows of Bt that are not a multiple of 16 bytes leave word by word: then from 2^24 on (one token, 672 x 14336
        // 21.0 / 23.4), and not where a quarter of the words that the workgroups take are beyond the row (25440 x 2464: 4 us
        // slower with blocks).
        const int64_t words = d_in / 32, signs = d_out * d_in;
        if (d_out % 128 == 0 ? signs > (int64_t)1 << 23 : signs >= (int64_t)1 << 24 && 4 * words >= 3 * ((words + 63) / 64 * 64)) {
            const dim3 grid((unsigned)((d_in / 32 + 63) / 64), (unsigned)((d_out + 127) / 128));
            hipLaunchKernelGGL(transpose_bits_blocks_kernel, grid, dim3(256), 0, stream, B_packed, Bt, (int)d_out, (int)d_in);
        } else {
            const dim3 grid((unsigned)((d_in / 32 + 3) / 4), (unsigned)((d_out + 63) / 64));
            hipLaunchKernelGGL(transpose_bits_kernel, grid, dim3(256), 0, stream, B_packed, Bt, (int)d_out, (int)d_in);
        }
        bits = Bt;
    }
    const int64_t n_tiles = (Nc + kGradBN - 1) / kGradBN;
    const dim3 grid((unsigned)(m_tiles * n_tiles));
    if (m_tiles == 0) {
        // no tokens: the reduction below writes zeros
    } else if (parts > 0) {
        const int rc = dtype == kBF16
            ? launch_grad_big<kBF16>(A, G, bits, partial, (int)M, (int)Nc, (int)Kc, (int)m_tiles, parts, stream)
            : launch_grad_big<kF16>(A, G, bits, partial, (int)M, (int)Nc, (int)Kc, (int)m_tiles, parts, stream);
        if (rc != 0) return rc;
    } else if (tune_value("grad_pipe", 1) != 0) {
        // the pipelined kernel is the default (grad_pipe=0: the two-workgroups-per-CU kernel)
        const int rc = dtype == kBF16
            ? launch_grad_tile_pipe<kBF16>(A, G, bits, partial, (int)M, (int)Nc, (int)Kc, (int)m_tiles, grid.x, stream)
            : launch_grad_tile_pipe<kF16>(A, G, bits, partial, (int)M, (int)Nc, (int)Kc, (int)m_tiles, grid.x, stream);
        if (rc != 0) return rc;
    } else if (dtype == kBF16)
        hipLaunchKernelGGL(grad_tile_kernel<kBF16>, grid, dim3(512), 0, stream, A, G, bits, partial, (int)M, (int)Nc,
                           (int)Kc, (int)m_tiles);
    else
        hipLaunchKernelGGL(grad_tile_kernel<kF16>, grid, dim3(512), 0, stream, A, G, bits, partial, (int)M, (int)Nc,
                           (int)Kc, (int)m_tiles);
    hipLaunchKernelGGL(grad_reduce_kernel, dim3((unsigned)((Nc + 63) / 64)), dim3(256), 0, stream,
                       (const float*)partial, grad, (int)Nc, (int)m_tiles * std::max(1, parts));
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace pdelta
