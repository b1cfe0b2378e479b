// Decode-shaped delta linear layer (1 to 64 tokens), d_in a multiple of 128: the arithmetic of pdelta_linear_skinny.hip (two
// accumulators, base and sign part, in the operands' own dtype) with all operands coming by direct loads into LDS.
//
// What bounds the register-staged kernel for batches: it reads X (61 tokens on 4096 inputs: 0.5 MB) once per 16 output
// rows and gets every 16 bytes into the MFMA's layout with four lane permutations, 80 per wave and 128 inputs at 64 tokens.
// A direct load puts them where one 16-byte LDS read finds them, and a workgroup takes 16, 32 or 48 rows, so X crosses the
// L2 a third as often.
//
// Work split: 8 waves, wave w with the units w, w + 8, ... of 128 inputs (the sums of the other decode kernels, bit for bit),
// LDS of its own and no barrier before the last sum.  A step is 64 inputs, whole 128-byte lines of every row (with 64-byte pieces 16 rows more cost a workgroup 4.5 us instead of 2.1: what
// a CU gets from memory is limited in requests, about 480 a us).  Several row tiles leave room for one stage per wave: a
// step goes to registers as a whole and the next is asked for before the products.  That beats more stages for four waves,
// whatever their number: alone on its SIMD a wave issues too slowly (61 tokens, 11008 x 4096, 48 rows: 29.4 us, and 22.9
// of them without any load in the loop).  Measured and dropped as well: waves that share X behind a barrier per step
// (28.7), the same with W_b asked for eight steps ahead (29.8).
//
// What is left is waiting.  Counters of 61 tokens, 11008 x 4096 bf16 (100.5 MB fetched, 1.04 of what has to be): matrix cores
// busy 24 % of the CU's cycles, vector ALUs 17 %, LDS 14 %; waves issue during 18 % of their life and spend 49 % on
// instructions that are under way.
//
// Calls in a row in a graph, weights changing, us, the kernels that took these calls before -> this one:
// bf16 row, 11008 x 4096, 61 tokens 46.9 -> 27.2, 24 tokens 33.4 -> 22.4, 16 tokens 23.3 -> 22.1; 4096 x 11008, 64 tokens
// 44.8 -> 36.9; 4096 x 4096, 64 tokens 18.8 -> 15.6, 24 tokens 13.6 -> 10.8.
#include <algorithm>
#include <type_traits>

#include "pdelta.h"
#include "pdelta_host.h"
#include "pdelta_lds_load.h"
#include "pdelta_skinny_tile.h"

namespace pdelta {

constexpr int kDmaBK = 64, kDmaUnitK = 128;           // inputs of a step and of a unit
constexpr int kDmaBufs = 4, kDmaWaves = 8;            // buffers of a unit's signs and scales; waves of a workgroup

// LDS bytes of one wave: DEPTH stages of X and W_b (rows of 128 bytes) and four buffers of what a unit of 128 inputs needs
// beside them: 16 bytes of signs per output row, in column mode v_col, blockwise four scales per output row.
constexpr int dma_wave_bytes(int axis, int mt, int nt, int depth)
{
    return depth * (mt + nt) * 2048 + kDmaBufs * (nt * 256 + (axis == 1 ? 256 : 0) + (axis == 2 ? nt * 256 : 0));
}

// One row tile: as many stages as the LDS of a CU holds, up to three.  A fourth brings nothing to a call by itself (16 tokens,
// 4096 x 4096 row: 9.0 us, 9.3 with two or four) and slows down calls on other streams (four streams, one token: 8.1 us a call,
// 8.9 with four, 7.6 with two, which cost a call by itself 0.2).  More
// tiles: one (32 rows, 24 tokens, 11008 x 4096: 25.9 us, 29.5 with two, which leave room for one workgroup a CU).
constexpr int dma_depth(int axis, int mt, int nt)
{
    if (nt > 1) return 1;
    int depth = 3;
    while (kDmaWaves * dma_wave_bytes(axis, mt, nt, depth) > 160 * 1024) --depth;
    return depth;
}

// s_waitcnt vmcnt(min(later, MAX) * EACH), later uniform
template <int EACH, int MAX>
__device__ __forceinline__ void wait_later(int later)
{
    if constexpr (MAX <= 0) wait_loads<0>();
    else if (later >= MAX) wait_loads<MAX * EACH>();
    else wait_later<EACH, MAX - 1>(later);
}

// MT tiles of 16 tokens, NT tiles of 16 output rows.
template <int XDT, int AXIS, int MT, int NT>
__global__ void __launch_bounds__(kDmaWaves * 64, 2)
linear_skinny_dma_kernel(const uint16_t* __restrict__ X, const uint16_t* __restrict__ W_b, const uint32_t* __restrict__ B_packed,
                         const uint16_t* __restrict__ v, void* __restrict__ Y, int M, int d_out, int d_in, int y_dtype,
                         int v_stride, int g_shift)
{
    constexpr int DEPTH = dma_depth(AXIS, MT, NT), WAVES = kDmaWaves;
    static_assert(DEPTH >= 1 && DEPTH <= 3 && NT <= 3, "a unit's signs would be overwritten too early");
    constexpr int XSTAGE = MT * 2048, STAGE = XSTAGE + NT * 2048, SIGNS = DEPTH * STAGE, SCALES = SIGNS + kDmaBufs * NT * 256,
                  WAVE_LDS = dma_wave_bytes(AXIS, MT, NT, DEPTH);
    constexpr int LOADS = 2 * (MT + NT);              // per step (signs and scales beside them)
    constexpr int SDT = AXIS == 0 ? XDT : kF16;       // dtype of the sign part's operands
    extern __shared__ __attribute__((aligned(16))) unsigned char dma_lds[];
    // (said to the compiler where it would otherwise keep a uniform value in vector registers)
    auto uniform = [](uint32_t x) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)x); };
    auto uniform_ptr = [&](const void* q) {
        const uint64_t u = (uint64_t)(uintptr_t)q;
        return (const char*)(uintptr_t)((uint64_t)uniform((uint32_t)(u >> 32)) << 32 | uniform((uint32_t)u));
    };
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int n = lane & 15, g = lane >> 4;
    const int n0 = blockIdx.x * (NT * 16);
    const int K = d_in;
    const uint32_t lds0 = uniform((uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)dma_lds + wave * WAVE_LDS);
    const unsigned char* const mine = dma_lds + wave * WAVE_LDS;

    // this wave's units are wave, wave + 8, ...; two steps each
    const int units = K / kDmaUnitK, n_steps = units > wave ? (units - wave + WAVES - 1) / WAVES * 2 : 0;
    auto input_of = [&](int s) { return uniform(((s >> 1) * WAVES + wave) * kDmaUnitK + (s & 1) * kDmaBK); };

    // a load covers 8 rows of 128 bytes; rows past the end repeat the last one
    const char* wbase = (const char*)(W_b + (int64_t)n0 * K);
    uint32_t xoff[2 * MT], woff[2 * NT], vgoff[NT];
    auto piece = [&](int q) { return (uint32_t)((lane & 7) ^ ((q & 1) * 4 + (lane >> 4))) * 16u; };
#pragma unroll
    for (int q = 0; q < 2 * MT; ++q) xoff[q] = (uint32_t)min(q * 8 + (lane >> 3), M - 1) * (uint32_t)K * 2u + piece(q);
#pragma unroll
    for (int q = 0; q < 2 * NT; ++q) woff[q] = (uint32_t)(min(n0 + q * 8 + (lane >> 3), d_out - 1) - n0) * (uint32_t)K * 2u + piece(q);
    // signs: lane = output row; scales: lane = 4 row + block of 32 inputs
    const char* sbase = (const char*)B_packed + (int64_t)n0 * (K >> 3);
    const uint32_t soff = (uint32_t)(min(n0 + lane, d_out - 1) - n0) * (uint32_t)(K >> 3);
    const uint16_t* vgbase = AXIS == 2 ? v + (int64_t)n0 * v_stride : v;
    if constexpr (AXIS == 2)
#pragma unroll
        for (int q = 0; q < NT; ++q) vgoff[q] = (uint32_t)(min(n0 + q * 16 + (lane >> 2), d_out - 1) - n0) * (uint32_t)v_stride;

    auto request = [&](int s, int slot) {
        const uint32_t kb = input_of(s);
        if ((s & 1) == 0) {                           // the unit's signs and scales
            const uint32_t buf = uniform((s >> 1) & (kDmaBufs - 1));
            if (lane < NT * 16) load_lds_16(uniform(lds0 + SIGNS + buf * (NT * 256)), soff, uniform_ptr(sbase + (kb >> 3)));
            if constexpr (AXIS == 1)
                if (lane < 16) load_lds_16(uniform(lds0 + SCALES + buf * 256), (kb + lane * 8) * 2u, uniform_ptr(v));
            if constexpr (AXIS == 2)
#pragma unroll
                for (int q = 0; q < NT; ++q)
                    load_lds_2(uniform(lds0 + SCALES + buf * (NT * 256)) + q * 256, (vgoff[q] + ((kb + (lane & 3) * 32) >> g_shift)) * 2u, uniform_ptr(vgbase));
        }
        const uint32_t stage = uniform(lds0 + slot * STAGE);
#pragma unroll
        for (int q = 0; q < 2 * NT; ++q) load_lds_16(stage + XSTAGE + q * 1024, woff[q], uniform_ptr(wbase + kb * 2u));
#pragma unroll
        for (int q = 0; q < 2 * MT; ++q) load_lds_16(stage + q * 1024, xoff[q], uniform_ptr((const char*)X + kb * 2u));
    };

    float4v accb[MT][NT], accs[MT][NT];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) accb[mt][nt] = accs[mt][nt] = (float4v){0.f, 0.f, 0.f, 0.f};
    float vr[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) vr[nt] = AXIS == 0 ? f16_bits_to_f32(v[min(n0 + nt * 16 + n, d_out - 1)]) : 1.0f;

    // lane (n, g) reads 16 bytes of row n: piece 4 j + g of its 128, stored at piece ^ ((n >> 1) & 7)
    const uint32_t frag = (uint32_t)(n * 128 + ((g ^ ((n >> 1) & 7)) * 16));
    uint32_t sign_bits = 0x80008000u, one2 = SDT == kBF16 ? 0x3F803F80u : 0x3C003C00u;
    asm volatile("" : "+v"(sign_bits), "+v"(one2));   // one literal per instruction
    uint4v x[2][MT], w[2][NT], vc[2];
    uint2v sw[2][NT];
    uint32_t vg[2][NT];
    auto read = [&](int s, int slot, auto parity, auto block) {
        constexpr int j = decltype(block)::value, par = decltype(parity)::value;
        const unsigned char* at = mine + slot * STAGE + (frag ^ (j * 64));
        const int buf = (s >> 1) & (kDmaBufs - 1);    // the step's two blocks are 2 par + j of the unit's four
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            if constexpr (j == 0) sw[par][nt] = *(const uint2v*)(mine + SIGNS + buf * (NT * 256) + (nt * 16 + n) * 16 + par * 8);
            if constexpr (AXIS == 2) vg[j][nt] = *(const uint32_t*)(mine + SCALES + buf * (NT * 256) + ((nt * 16 + n) * 4 + par * 2 + j) * 4);
            w[j][nt] = *(const uint4v*)(at + XSTAGE + nt * 2048);
        }
        if constexpr (AXIS == 1) vc[j] = *(const uint4v*)(mine + SCALES + buf * 256 + par * 128 + j * 64 + g * 16);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) x[j][mt] = *(const uint4v*)(at + mt * 2048);
    };
    auto multiply = [&](auto parity, auto block) {
        constexpr int j = decltype(block)::value;
        uint4v sg[NT];
#pragma unroll
        for (int nt = 0; nt < NT; ++nt) {
            const uint32_t minus = ~(sw[decltype(parity)::value][nt][j] >> (g * 8)) & 0xFFu;
            uint32_t y = minus | (minus << 15);       // bit 2p at 2p, bit 2p + 1 at 2p + 16
            asm("" : "+v"(y));                        // (else y and its shifts become full multiplications)
#pragma unroll
            for (int p = 0; p < 4; ++p) sg[nt][p] = ((y << (15 - 2 * p)) & sign_bits) | one2;
            if constexpr (AXIS == 2) sg[nt] = signs_times_scale(sg[nt], vg[j][nt]);
        }
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
            uint4v xs = x[j][mt];
            if constexpr (AXIS == 1) xs = scale_x<XDT>(x[j][mt], vc[j]);
            if constexpr (AXIS == 2) xs = x_as_f16<XDT>(x[j][mt]);
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) {
                accb[mt][nt] = mfma16<XDT>(x[j][mt], w[j][nt], accb[mt][nt]);
                accs[mt][nt] = mfma16<SDT>(xs, sg[nt], accs[mt][nt]);
            }
        }
    };

    if (n_steps > 0) {                                // wave-uniform; the barrier is below
        using B0 = std::integral_constant<int, 0>;
        using B1 = std::integral_constant<int, 1>;
#pragma unroll
        for (int d = 0; d < DEPTH; ++d)
            if (d < n_steps) request(d, d);
        if constexpr (DEPTH > 1) {
            wait_later<LOADS, DEPTH - 1>(min(n_steps, DEPTH) - 1);
            read(0, 0, B0{}, B0{});
        }
        int slot = 0;
        auto step = [&](int s, auto parity, auto other) {
            if constexpr (DEPTH == 1) {               // one stage: all of the step goes to registers, then the next is asked for
                wait_loads<0>();
                read(s, 0, parity, B0{});
                read(s, 0, parity, B1{});
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                if (s + 1 < n_steps) request(s + 1, 0);
                multiply(parity, B0{});
                multiply(parity, B1{});
                __builtin_amdgcn_sched_barrier(0);
                return;
            }
            const int next = __builtin_amdgcn_readfirstlane(slot + 1 == DEPTH ? 0 : slot + 1);
            read(s, slot, parity, B1{});
            __builtin_amdgcn_sched_barrier(0);
            multiply(parity, B0{});
            __builtin_amdgcn_sched_barrier(0);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");      // step s is in registers, its stage is free
            if (s + DEPTH < n_steps) request(s + DEPTH, slot);
            if (s + 1 < n_steps) {
                wait_later<LOADS, DEPTH - 1>(min(n_steps - 2 - s, DEPTH - 1));       // the steps asked for after s + 1
                read(s + 1, next, other, B0{});
            }
            __builtin_amdgcn_sched_barrier(0);
            multiply(parity, B1{});
            __builtin_amdgcn_sched_barrier(0);
            slot = next;
        };
        for (int s = 0; s < n_steps; s += 2) {
            step(s, B0{}, B1{});
            step(s + 1, B1{}, B0{});
        }
    }

    // each wave's sums in its own LDS (all its loads have been waited for and read), then all waves'
    float* red = (float*)mine;                        // [MT][NT][4][64]
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int r = 0; r < 4; ++r) red[((mt * NT + nt) * 4 + r) * 64 + lane] = accb[mt][nt][r] + vr[nt] * accs[mt][nt][r];
    __syncthreads();
    for (int idx = threadIdx.x; idx < MT * NT * 256; idx += WAVES * 64) {
        const int oc = idx % (NT * 16), t = idx / (NT * 16), oo = n0 + oc;
        const int at = (((t >> 4) * NT + (oc >> 4)) * 4 + (t & 3)) * 64 + ((t >> 2) & 3) * 16 + (oc & 15);
        float sum = 0.f;
#pragma unroll
        for (int k = 0; k < WAVES; ++k) sum += *(const float*)(dma_lds + k * WAVE_LDS + at * 4);
        if (t < M && oo < d_out) {
            const int64_t yi = (int64_t)t * d_out + oo;
            if (y_dtype == kF32) store_y<kF32>(Y, yi, sum);
            else if (y_dtype == kBF16) store_y<kBF16>(Y, yi, sum);
            else store_y<kF16>(Y, yi, sum);
        }
    }
}

template <int XDT, int AXIS, int MT, int NT>
static int launch_dma(const void* X, const void* W_b, const uint32_t* B_packed, const uint16_t* v, void* Y, int64_t M,
                      int64_t d_out, int64_t d_in, int y_dtype, int v_stride, int g_shift, hipStream_t stream)
{
    constexpr int wave_lds = dma_wave_bytes(AXIS, MT, NT, dma_depth(AXIS, MT, NT)), lds = kDmaWaves * wave_lds;
    static_assert(wave_lds >= MT * NT * 1024 && lds <= 160 * 1024, "LDS of a workgroup");
    auto kernel = linear_skinny_dma_kernel<XDT, AXIS, MT, NT>;
    static unsigned lds_opted_in = 0;                 // per template instance: one kernel
    if (opt_in_dynamic_lds((const void*)kernel, lds, &lds_opted_in) != 0) return -1;
    hipLaunchKernelGGL(kernel, dim3((unsigned)((d_out + NT * 16 - 1) / (NT * 16))), dim3(kDmaWaves * 64), lds, stream, (const uint16_t*)X,
                       (const uint16_t*)W_b, B_packed, v, Y, (int)M, (int)d_out, (int)d_in, y_dtype, v_stride, g_shift);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

template <int XDT, int AXIS>
static int launch_dma_tokens(const void* X, const void* W_b, const uint32_t* B_packed, const uint16_t* v, void* Y, int64_t M,
                             int64_t d_out, int64_t d_in, int y_dtype, int v_stride, int g_shift, int nt, hipStream_t stream)
{
    const int mt = (int)((M + 15) / 16);
#define PDELTA_GO(MT, NT) \
    return launch_dma<XDT, AXIS, MT, NT>(X, W_b, B_packed, v, Y, M, d_out, d_in, y_dtype, v_stride, g_shift, stream)
#define PDELTA_ROWS(MT)           \
    {                             \
        if (nt == 1) PDELTA_GO(MT, 1); \
        if (nt == 2) PDELTA_GO(MT, 2); \
        PDELTA_GO(MT, 3);         \
    }
    if (mt == 1) PDELTA_ROWS(1)
    if (mt == 2) PDELTA_ROWS(2)
    if (mt == 3) PDELTA_ROWS(3)
    PDELTA_ROWS(4)
#undef PDELTA_ROWS
#undef PDELTA_GO
}

int launch_linear_skinny_dma(int x_dtype, int y_dtype, int axis, const void* X, const void* W_b, const uint32_t* B_packed,
                             const uint16_t* v, void* Y, int64_t M, int64_t d_out, int64_t d_in, int v_stride, int g_shift,
                             int rows, hipStream_t stream)
{
#define PDELTA_GO(XDT, AXIS) return launch_dma_tokens<XDT, AXIS>(X, W_b, B_packed, v, Y, M, d_out, d_in, y_dtype, v_stride, g_shift, rows, stream)
    if (x_dtype == kBF16) {
        if (axis == 0) PDELTA_GO(kBF16, 0);
        if (axis == 1) PDELTA_GO(kBF16, 1);
        PDELTA_GO(kBF16, 2);
    }
    if (axis == 0) PDELTA_GO(kF16, 0);
    if (axis == 1) PDELTA_GO(kF16, 1);
    PDELTA_GO(kF16, 2);
#undef PDELTA_GO
}

}  // namespace pdelta
