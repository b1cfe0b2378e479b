// Prefill-shaped delta linear layer, d_in a multiple of 128: the arithmetic of pdelta_linear_gemm.hip
// (W_hat = fp16(W_b +- v), X as fp16, fp32 sums in the order of d_in) on tiles of 256 tokens x 256 output
// rows x 64 inputs, 8 waves of 128 x 64 outputs, with all global traffic as direct loads into LDS.
//
// What bounds it, found by taking parts out in working builds (2048 x 8192 x 4096 fp16, one full round of 256 tiles, 131 us
// against 152 for the 256 x 128 register-staged kernel): MFMAs, fragment reads and conversion alone 114 us
// (the matrix cores' own ceiling with random operands is 81), everything but the MFMAs 91.  The
// latter is the L1's request rate, about one request every two cycles whether it is for 64 or 128 bytes;
// hence the tile (half the operand bytes per product of a 256 x 128 tile), whole 128-byte lines per row and
// step, and sign words fetched for four steps at a time: with 32-input steps and one sign word per row
// and step, a third of all requests were for signs and the same tile took 146 us.
//
// Two LDS stages.  A wave converts what it has itself loaded, in place: W_b becomes W_hat, bf16 X becomes
// fp16; wave-private, so only its own loads have to be waited for.  One barrier per step, three quarters
// into it: by then a wave has read its last fragments of step s and converted its part of step s+1, so the
// barrier publishes step s+1 and frees the stage of step s, which is requested at once for step s+2; the
// last quarter's MFMAs run while the first fragments of step s+1 are read.
//
// With W_b in HBM (a program's other layers ran in between) two stages are too little lead for the first
// reader of a line, so each workgroup also touches its share of the W_b lines kBigFar steps ahead (touch_rows): 2048 x
// 11008 x 4096 bf16 on changing inputs 237 -> 227 us (236 for the 256 x 128 kernel), 777 x 4096 x 11008
// blockwise 131 -> 126 (253); on inputs that stay cached it is within 2 %.  Touching the lines of both
// operands from every workgroup costs more than it gives (the L1's request rate again).
//
// LDS rows are 128 bytes, unpadded as direct loads require; the 16-byte piece p of row r holds inputs
// 8 (p ^ ((r >> 1) & 7)) .. +7, so that 16 consecutive rows of one fragment read touch all 64 banks once.
// The permutation is applied by choosing which 16 bytes each lane loads.
//
// Work split: tiles that fill whole rounds of the 256 CUs are computed in one go; the remaining ones, in the
// calls that may split, in parts of d_in, whose sums a second kernel adds in the order of d_in.
// Workgroup w runs on XCD w % 8; each XCD takes a contiguous range of the whole tiles (token tiles of one
// output-row tile first, so that its CUs share W_b panels in its L2), then one of the parts.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "pdelta_gemm_tile.h"
#include "pdelta_host.h"
#include "pdelta_lds_load.h"

namespace pdelta {

constexpr int kBigTile = 256, kBigBK = 64, kBigUnitK = 128, kBigFar = 4;   // parts of d_in: multiples of 128 inputs
constexpr int kBigXB = kBigTile * kBigBK * 2, kBigStage = 2 * kBigXB;   // bytes of X (of W_b) and of a stage
// behind the two stages, per wave: the sign words of its 32 rows for four steps (1 KB); the four steps' v_col
// (column mode, 1 KB) or the step's scales of its rows (blockwise, 256 B)
constexpr int kBigSigns = 2 * kBigStage, kBigScales = kBigSigns + 8 * 1024, kBigTouch = kBigScales + 8 * 1024, kBigLds = kBigTouch + 8 * 256;
constexpr size_t kPartBytes = (size_t)kBigTile * kBigTile * 4;      // fp32 partial sums of one tile

// Rows of a W_b tile that each of the workgroups sharing it touches ahead of its loads, and the lanes of a wave that
// do so.  All rows are covered, except by a workgroup that has the tile to itself: each line is then loaded only
// once anyway, and 64 of the rows are better than all (256 x 14336 x 4096 bf16 63 against 65 us).  With 64 rows also
// for two and three sharers, 500 x 4096 x 11008 took 81 instead of 79.5 us and 700 x 11008 x 4096 139 instead of 133.5.
constexpr __host__ __device__ int touch_rows(int sharers) { return (kBigTile + sharers - 1) / sharers; }
constexpr __host__ __device__ int touch_lanes(int sharers) { return sharers == 1 ? 8 : (touch_rows(sharers) + 7) / 8; }
constexpr bool touch_covers_the_tile(int sharers)
{
    return sharers > 8 || (8 * touch_lanes(sharers) >= touch_rows(sharers) && sharers * touch_rows(sharers) >= kBigTile &&
                           touch_lanes(sharers) <= 64 && touch_covers_the_tile(sharers + 1));
}
static_assert(touch_covers_the_tile(2), "a line that is not touched is waited for by its first reader");

// x ^ C.  HERE: computed where it stands.  As ordinary expressions the LDS addresses of the loop are all kept in
// registers, up to 20 of them, and for fp16 with column or blockwise scales there are not enough (accumulators, two
// sets of fragments and raw weights take 200 of the 256): 5 and 11 were spilled and reloaded between the MFMAs, each
// reload waiting for the direct loads before it.  fp16, column / blockwise, with and without the spills: 2048 x 8192 x
// 4096 154 -> 143 / 165 -> 148 us, 777 x 4096 x 11008 blockwise 137 -> 123.  bf16 reads the raw weights when fewer
// fragments are held, and with row scales there is no scale to fetch.
template <bool HERE, int C>
__device__ __forceinline__ uint32_t xor_at(uint32_t x)
{
    if constexpr (!HERE) return x ^ (uint32_t)C;
    uint32_t r;
    asm volatile("v_xor_b32 %0, %1, %2" : "=v"(r) : "n"(C), "v"(x));
    return r;
}

template <int WDT, int AXIS>
__global__ void __launch_bounds__(512, 2)
linear_gemm_big_kernel(const uint16_t* __restrict__ X, const uint16_t* __restrict__ W_b,
                       const uint32_t* __restrict__ B_packed, const uint16_t* __restrict__ v,
                       void* __restrict__ Y, float* __restrict__ partial, int M, int d_out, int d_in, int y_dtype,
                       int m_tiles, int whole, int split, int parts, int v_stride, int g_shift)
{
    constexpr int FM = 4, FN = 2;                     // a wave owns 128 tokens x 64 output rows
    constexpr bool HERE = WDT != kBF16 && AXIS != 0;  // see xor_at
    extern __shared__ __attribute__((aligned(16))) unsigned char dma_smem[];

    // tile and part of this workgroup (see the map in the header comment)
    const int K = d_in;
    const int xcd = blockIdx.x % kXcds;
    const int whole_per = (whole + kXcds - 1) / kXcds;
    int tile, k_first = 0, k_end = K / kBigUnitK, unit = -1;
    if ((int)blockIdx.x < whole_per * kXcds) {
        const int j = (int)blockIdx.x / kXcds;
        tile = xcd * whole_per + j;
        if (tile >= whole) return;                    // whole workgroup
    } else {
        const int units = split * parts, per = (units + kXcds - 1) / kXcds;
        const int j = ((int)blockIdx.x - whole_per * kXcds) / kXcds;
        unit = xcd * per + j;
        if (unit >= units) return;                    // whole workgroup
        const int part = unit / split;
        tile = whole + unit % split;
        k_first = (int)((int64_t)k_end * part / parts);
        k_end = (int)((int64_t)k_end * (part + 1) / parts);
    }
    const int m0 = (tile % m_tiles) * kBigTile, n0 = (tile / m_tiles) * kBigTile;
    const int n_steps = (k_end - k_first) * (kBigUnitK / kBigBK);     // even, at least 2
    const int kb0 = k_first * kBigUnitK, kb_end = k_end * kBigUnitK;

    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int wm = wave >> 2, wn = wave & 3;
    const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)dma_smem;

    // One load instruction covers 8 tile rows of 128 bytes, a wave loads 32 rows of each operand; rows
    // past the end of X or W_b repeat the last one (they only feed outputs that are never stored).
    const char* xbase = (const char*)(X + (int64_t)m0 * K + kb0);
    const char* wbase = (const char*)(W_b + (int64_t)n0 * K + kb0);
    uint32_t chunk[2], xoff[4], woff[4], vrow[4];
#pragma unroll
    for (int q = 0; q < 2; ++q) chunk[q] = (uint32_t)((lane & 7) ^ (q * 4 + (lane >> 4)));
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int r = wave * 32 + q * 8 + (lane >> 3);
        xoff[q] = (uint32_t)(min(m0 + r, M - 1) - m0) * (uint32_t)K * 2u + chunk[q & 1] * 16u;
        const int row = min(n0 + r, d_out - 1) - n0;
        woff[q] = (uint32_t)row * (uint32_t)K * 2u + chunk[q & 1] * 16u;
        if constexpr (AXIS == 0) vrow[q] = (uint32_t)v[n0 + row] * 0x10001u;
    }
    // lanes 0-31: sign words of the wave's rows for two steps, lanes 32-63 for the next two
    const int srow = min(n0 + wave * 32 + (lane & 31), d_out - 1) - n0;
    const char* sbase = (const char*)B_packed + (int64_t)n0 * (K >> 3) + (kb0 >> 3);
    const uint32_t soff = (uint32_t)srow * (uint32_t)(K >> 3) + (lane >> 5) * 16u;
    const uint16_t* vgbase = v + (int64_t)n0 * v_stride;
    const uint32_t vgoff = (uint32_t)srow * (uint32_t)v_stride;
    const int g_step = AXIS == 2 && g_shift < 31 ? max(1 << g_shift, kBigBK) : 0;   // 0: one scale for all of d_in

    // signs and scales of step s (if it is the first that they serve), then W_b, then X
    auto request = [&](int s, uint32_t stage) {
        const int rel = s * kBigBK, kb = kb0 + rel;
        if ((s & 3) == 0) {                           // never past d_in: a short last group repeats its first half
            load_lds_16(lds0 + kBigSigns + wave * 1024, kb + 128 < kb_end ? soff : soff - (lane >> 5) * 16u, sbase + (rel >> 3));
            if constexpr (AXIS == 1)
                load_lds_16(lds0 + kBigScales + wave * 1024, (uint32_t)min(kb + (lane & 31) * 8, kb_end - 8) * 2u, v);
        }
        if constexpr (AXIS == 2) {
            if (s == 0 || (g_step != 0 && (kb & (g_step - 1)) == 0))
                load_lds_2(lds0 + kBigScales + wave * 1024, (vgoff + (uint32_t)((kb + (lane >> 5) * 32) >> g_shift)) * 2u, vgbase);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) load_lds_16(lds0 + stage + kBigXB + (wave * 4 + q) * 1024, woff[q], wbase + (int64_t)rel * 2);
#pragma unroll
        for (int q = 0; q < 4; ++q) load_lds_16(lds0 + stage + (wave * 4 + q) * 1024, xoff[q], xbase + (int64_t)rel * 2);
    };

    // L2 prefetch of W_b, kBigFar steps ahead: the workgroups of one output-row tile on an XCD share its 256
    // rows, the first lanes of each wave touch one 128-byte line each.  (The data goes to LDS that nobody reads.)
    const int sharers = min(m_tiles, 8), lanes = touch_lanes(sharers);
    const int trow = min((tile % m_tiles % sharers) * touch_rows(sharers) + wave * lanes + lane, kBigTile - 1);
    const uint32_t poff = (uint32_t)(min(n0 + trow, d_out - 1) - n0) * (uint32_t)K * 2u;
    auto prefetch = [&](int s) {
        if (lane < lanes) load_lds_4(lds0 + kBigTouch + wave * 256, poff, wbase + (int64_t)min(s + kBigFar, n_steps - 1) * (kBigBK * 2));
    };

    // In place: the wave's own pieces of W_b -> W_hat, of bf16 X -> fp16.
    uint4v raw[4], wvec[2];
    uint32_t sbyte[4], wscale[4];
    // sign byte and scale of the wave's rows lane / 8 + 8 q, LDS piece lane % 8
    const uint32_t sign0 = (uint32_t)(lane >> 3) * 16 + chunk[0], scale0 = ((chunk[0] >> 2) * 32 + (uint32_t)(lane >> 3)) * 4;
    auto fetch_w = [&](int s, uint32_t stage) {
        const unsigned char* signs = dma_smem + kBigSigns + wave * 1024 + ((s >> 1) & 1) * 512 + (s & 1) * 8;
        const unsigned char* scales = dma_smem + kBigScales + wave * 1024;
        const uint32_t sign_at[2] = {sign0, xor_at<HERE, 4>(sign0)};      // chunk[1] = chunk[0] ^ 4
        uint32_t scale_at[2] = {scale0, 0};
        if constexpr (AXIS == 2) scale_at[1] = xor_at<HERE, 128>(scale0);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            raw[q] = *(const uint4v*)(dma_smem + stage + kBigXB + (wave * 4 + q) * 1024 + lane * 16);
            sbyte[q] = signs[q * 128 + sign_at[q & 1]];
            if constexpr (AXIS == 2) wscale[q] = *(const uint16_t*)(scales + q * 32 + scale_at[q & 1]);
        }
        if constexpr (AXIS == 1) {
#pragma unroll
            for (int q = 0; q < 2; ++q) wvec[q] = *(const uint4v*)(scales + (s & 3) * 128 + chunk[q] * 16);
        }
    };
    auto convert_w = [&](uint32_t stage) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const uint32_t neg = ~sbyte[q] & 0xFFu;
            uint32_t y = neg | (neg << 15);           // bit 2p + 1 at 2p + 16
            asm("" : "+v"(y));                        // (else y and its shifts become full multiplications)
            const uint32_t vv = AXIS == 2 ? wscale[q] | (wscale[q] << 16) : (AXIS == 0 ? vrow[q] : 0u);
            const uint4v w16 = to_f16x8<WDT>(raw[q]);
            uint4v r;
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                const uint32_t vp = AXIS == 1 ? wvec[q & 1][p] : vv, wp = w16[p];
                const uint32_t sv = ((y << (15 - 2 * p)) & 0x80008000u) ^ vp;     // -v where the bit is set
                r[p] = as_u32(as_half2(wp) + as_half2(sv));
            }
            *(uint4v*)(dma_smem + stage + kBigXB + (wave * 4 + q) * 1024 + lane * 16) = r;
        }
    };
    auto fetch_x = [&](uint32_t stage) {
#pragma unroll
        for (int q = 0; q < 4; ++q) raw[q] = *(const uint4v*)(dma_smem + stage + (wave * 4 + q) * 1024 + lane * 16);
    };
    auto convert_x = [&](uint32_t stage) {
#pragma unroll
        for (int q = 0; q < 4; ++q) *(uint4v*)(dma_smem + stage + (wave * 4 + q) * 1024 + lane * 16) = to_f16x8<kBF16>(raw[q]);
    };

    float16v acc[FM][FN];
#pragma unroll
    for (int f = 0; f < FM; ++f)
#pragma unroll
        for (int h = 0; h < FN; ++h)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[f][h][r] = 0.f;

    // this lane's piece of 16 inputs ks is at byte frag ^ (32 ks)
    const uint32_t frag = (uint32_t)((lane & 31) * 128 + (((lane >> 5) ^ ((lane >> 1) & 7)) * 16));
    half8 a[2][FM], b[2][FN];
    auto read_frags = [&](uint32_t stage, auto step16) {
        constexpr int ks = decltype(step16)::value;
        const uint32_t piece = xor_at<HERE, ks * 32>(frag);
        const unsigned char* xa = dma_smem + stage + wm * 128 * 128 + piece;
        const unsigned char* wa = dma_smem + stage + kBigXB + wn * 64 * 128 + piece;
#pragma unroll
        for (int h = 0; h < FN; ++h) b[ks & 1][h] = *(const half8*)(wa + h * 32 * 128);
#pragma unroll
        for (int f = 0; f < FM; ++f) a[ks & 1][f] = *(const half8*)(xa + f * 32 * 128);
    };
    auto multiply = [&](int ks) {
#pragma unroll
        for (int f = 0; f < FM; ++f)
#pragma unroll
            for (int h = 0; h < FN; ++h)
                acc[f][h] = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[ks & 1][f], b[ks & 1][h], acc[f][h], 0, 0, 0);
    };

    request(0, 0);
    wait_loads<0>();
    fetch_w(0, 0);
    convert_w(0);
    if constexpr (WDT == kBF16) { fetch_x(0); convert_x(0); }
    lds_barrier();
    request(1, kBigStage);
    read_frags(0, std::integral_constant<int, 0>{});

    // Step s; REQ: request step s + 2, MORE: there is a step s + 1.  The fences keep the LDS reads above
    // the MFMAs (left alone, the compiler sinks them below) and the conversion between them.
    auto step = [&](int s, uint32_t cur, uint32_t nxt, auto req, auto more) {
        constexpr bool REQ = decltype(req)::value, MORE = decltype(more)::value;
        read_frags(cur, std::integral_constant<int, 1>{});
        __builtin_amdgcn_sched_barrier(0);
        multiply(0);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (MORE) {
            if constexpr (WDT == kBF16) wait_loads<4>(); else wait_loads<0>();    // (the last four are X)
            if constexpr (WDT == kBF16) fetch_w(s + 1, nxt);
        }
        if constexpr (REQ && WDT != kBF16) prefetch(s);
        read_frags(cur, std::integral_constant<int, 2>{});
        if constexpr (MORE && WDT != kBF16) fetch_w(s + 1, nxt);
        __builtin_amdgcn_sched_barrier(0);
        multiply(1);
        if constexpr (MORE && WDT == kBF16) { convert_w(nxt); interleave<FM * FN, 13>(); }
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (MORE && WDT == kBF16) { wait_loads<0>(); fetch_x(nxt); }
        if constexpr (REQ && WDT == kBF16) prefetch(s);
        read_frags(cur, std::integral_constant<int, 3>{});
        __builtin_amdgcn_sched_barrier(0);
        multiply(2);
        if constexpr (MORE && WDT == kBF16) { convert_x(nxt); interleave<FM * FN, 6>(); }
        if constexpr (MORE && WDT != kBF16) { convert_w(nxt); interleave<FM * FN, 7>(); }
        __builtin_amdgcn_sched_barrier(0);
        lds_barrier();
        if constexpr (MORE) read_frags(nxt, std::integral_constant<int, 0>{});
        if constexpr (REQ) request(s + 2, cur);
        __builtin_amdgcn_sched_barrier(0);
        multiply(3);
        __builtin_amdgcn_sched_barrier(0);
    };
    int s = 0;
    for (; s + 2 < n_steps; s += 2) {
        step(s, 0, kBigStage, std::true_type{}, std::true_type{});
        step(s + 1, kBigStage, 0, std::true_type{}, std::true_type{});
    }
    step(s, 0, kBigStage, std::false_type{}, std::true_type{});
    step(s + 1, kBigStage, 0, std::false_type{}, std::false_type{});

    if (unit >= 0) {                                  // a part of d_in: the sums as they are
        float4v* out = (float4v*)(partial + (int64_t)unit * (kBigTile * kBigTile)) + wave * (FM * FN * 4 * 64) + lane;
#pragma unroll
        for (int f = 0; f < FM; ++f)
#pragma unroll
            for (int h = 0; h < FN; ++h)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    out[((f * FN + h) * 4 + r) * 64] =
                        (float4v){acc[f][h][4 * r], acc[f][h][4 * r + 1], acc[f][h][4 * r + 2], acc[f][h][4 * r + 3]};
        return;
    }
    // (the last barrier came after the last fragment read: the stages are free)
    store_wave_tile<FM>(acc, (uint16_t*)dma_smem + wave * 32 * kGemmLDK, Y, y_dtype, m0 + wm * 128, n0 + wn * 64, M, d_out, lane);
}

// Sums of the parts of the split tiles, in the order of d_in, and their outputs: a wave takes the
// 32 tokens x 64 outputs (wave w, block f) of a tile.
__global__ void __launch_bounds__(256)
linear_gemm_sum_kernel(const float* __restrict__ partial, void* __restrict__ Y, int M, int d_out, int y_dtype,
                       int m_tiles, int whole, int split, int parts)
{
    __shared__ __attribute__((aligned(16))) uint16_t region[4 * 32 * kGemmLDK];
    const int lane = threadIdx.x & 63, f = threadIdx.x >> 6;
    const int t = blockIdx.x >> 3, w = blockIdx.x & 7, tile = whole + t;
    const int tok0 = (tile % m_tiles) * kBigTile + (w >> 2) * 128 + f * 32;
    const int o0 = (tile / m_tiles) * kBigTile + (w & 3) * 64;
    if (tok0 >= M || o0 >= d_out) return;             // wave-uniform, no barrier follows
    float16v acc[1][2];
    const float4v* in = (const float4v*)partial + ((int64_t)t * 8 + w) * (4 * 2 * 4 * 64) + f * (2 * 4 * 64) + lane;
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[0][h][r] = 0.f;
    for (int p = 0; p < parts; ++p, in += (int64_t)split * (kBigTile * kBigTile / 4)) {
        float4v x[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) x[i] = in[i * 64];
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[0][i >> 2][(i & 3) * 4 + e] += x[i][e];
    }
    store_wave_tile<1>(acc, region + f * 32 * kGemmLDK, Y, y_dtype, tok0, o0, M, d_out, lane);
}

template <int WDT, int AXIS>
static int launch_big(const void* X, const void* W_b, const uint32_t* B_packed, const uint16_t* v, void* Y, int64_t M,
                      int64_t d_out, int64_t d_in, int y_dtype, int v_stride, int g_shift, void* workspace,
                      BigSplit sp, hipStream_t stream)
{
    constexpr size_t lds = kBigLds;                   // 149,504 bytes
    const int m_tiles = (int)((M + kBigTile - 1) / kBigTile);
    auto kernel = linear_gemm_big_kernel<WDT, AXIS>;
    static unsigned lds_opted_in = 0;                 // per template instance: one kernel
    if (opt_in_dynamic_lds((const void*)kernel, (int)lds, &lds_opted_in) != 0) return -1;
    const int units = sp.split * sp.parts;
    const int blocks = ((sp.whole + kXcds - 1) / kXcds + (units + kXcds - 1) / kXcds) * kXcds;
    hipLaunchKernelGGL(kernel, dim3((unsigned)blocks), dim3(512), lds, stream, (const uint16_t*)X, (const uint16_t*)W_b,
                       B_packed, v, Y, (float*)workspace, (int)M, (int)d_out, (int)d_in, y_dtype, m_tiles, sp.whole, sp.split,
                       sp.parts, v_stride, g_shift);
    if (sp.split > 0)
        hipLaunchKernelGGL(linear_gemm_sum_kernel, dim3((unsigned)sp.split * 8), dim3(256), 0, stream, (const float*)workspace,
                           Y, (int)M, (int)d_out, y_dtype, m_tiles, sp.whole, sp.split, sp.parts);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

// Which calls run here, and how many tiles are split.  Both sides are priced with what was measured
// (us, 256 CUs, steps of 64 inputs): here a step takes 1.75 (fp16) or 1.95 (bf16), a call 8 beside its
// steps, a split 8 more for its second launch and 0.06 per part for the sums that it writes and reads;
// the 256 x 128 kernel takes 1.0 / 1.08 a step and 15 a call, the 64 x 64 kernels 3 a call and 0.29 / 0.31 a step, 0.05
// more with column or blockwise scales (128 x 3072 x 8192 fp16: 44, 48 and 51 there, 42-44 here in 16 parts) and 0.045 more
// when every CU has a tile; above one tile per CU 0.3 for each of the tiles of the busiest CU and 0.15 for what they are
// together, 0.05-0.15 more with other scales or bf16 (of 1640 calls within 1 % of the best choice on average; a price that
// grows with the tiles alone left 140 x 6656 x 8192 bf16, 312 tiles, there: 90, here 62 in 8 parts).  Against the 64 x 64 kernels a split pays 0.1 more per part: it
// has few tiles there, and a wave of the second launch reads the parts of its outputs one after another.  bf16, changing
// inputs, this kernel against the others: 2048 x 11008 x 4096 (88 of 344 tiles in 2 parts) 223-230 against 230-237, 777 x
// 4096 x 11008 blockwise (64 tiles in 4 parts) 127 against 254, 1024 x 4096 x 4096 60 against 87, 256 x 512 x 8192 (2 tiles
// in 16 parts) 36 against 43, 448 x 960 x 8192 fp16 blockwise (8 tiles in 16 parts) 38 against 45.5.  Below the line: 256 x
// 1024 x 4096 (4 tiles in 16 parts) fp16 35 against 23, 402 x 384 x 5760 fp16 31 against 23, 251 x 4096 x 4096 32 against 25.
BigSplit linear_gemm_big_split(int64_t M, int64_t d_out, int64_t d_in, int x_dtype, int axis, bool split_allowed)
{
    const BigSplit none{0, 0, 0};
    const int forced = tune_value("gemm_big", -1);    // 0: never; n > 0: in n parts (1: whole tiles only)
    if (d_in % kBigUnitK != 0 || forced == 0) return none;
    if (forced < 0 && (tune_value("gemm_small", -1) >= 0 || tune_value("gemm_pipe", -1) >= 0 || tune_value("gemm_bm", -1) >= 0))
        return none;                                  // another kernel is asked for
    const int64_t tiles = ((M + kBigTile - 1) / kBigTile) * ((d_out + kBigTile - 1) / kBigTile);
    if (tiles > (1 << 24)) return none;
    const int rest = (int)(tiles % 256), whole = (int)(tiles - rest);
    const double n = (double)(d_in / kBigBK), step = x_dtype == kBF16 ? 1.95 : 1.75;
    auto fits = [&](int p) { return split_allowed && p <= d_in / kBigUnitK && rest * p <= 256; };
    if (forced == 1 || (forced > 1 && !fits(forced))) return BigSplit{(int)tiles, 0, 1};
    if (forced > 1) return rest > 0 ? BigSplit{whole, rest, forced} : BigSplit{whole, 0, 1};
    double best = 8 + (double)((tiles + 255) / 256) * n * step;
    BigSplit sp{(int)tiles, 0, 1};
    for (int p = 2; p <= 16 && rest > 0 && fits(p); ++p) {
        const double t = 16 + ((double)(whole / 256) * n + std::ceil(n / p / 2) * 2) * step + 0.06 * rest * p;
        if (t < best) { best = t; sp = BigSplit{whole, rest, p}; }
    }
    const int64_t tiles128 = ((M + 255) / 256) * ((d_out + kGemmBN - 1) / kGemmBN);
    const int64_t tiles64 = ((M + 63) / 64) * ((d_out + 63) / 64);
    if (tiles128 <= 128) {
        const bool bf16 = x_dtype == kBF16;
        const double row = bf16 ? 0.31 : 0.29, each = (double)tiles64 / 256, most = std::ceil(each);
        const double over = axis == 0 ? (bf16 ? 0.05 : 0) : axis == 1 ? (bf16 ? 0.12 : 0.05) : (bf16 ? 0.15 : 0.1);
        const double small = 3 + n * (tiles64 <= 256 ? (axis == 0 ? row : row + 0.05) + 0.045 * each
                                                     : 0.3 * most + 0.15 * (each - (most - 1)) + over);
        return best + (sp.split > 0 ? 0.1 * sp.parts : 0) < small ? sp : none;
    }
    const double pipe = 15 + n * (double)((tiles128 + 255) / 256) * (x_dtype == kBF16 ? 1.08 : 1.0);
    return best < 0.97 * pipe ? sp : none;
}

size_t linear_gemm_workspace_bytes(int64_t M, int64_t d_out, int64_t d_in, int x_dtype)
{
    const BigSplit sp = linear_gemm_big_split(M, d_out, d_in, x_dtype, 2, true);       // row calls split in some of these cases only
    return (size_t)sp.split * sp.parts * kPartBytes;
}

int launch_linear_gemm_big(int x_dtype, int y_dtype, int axis, const void* X, const void* W_b,
                           const uint32_t* B_packed, const uint16_t* v, void* Y, int64_t M, int64_t d_out,
                           int64_t d_in, int v_stride, int g_shift, void* workspace, BigSplit sp, hipStream_t stream)
{
#define PDELTA_GO(WDT, AXIS) \
    return launch_big<WDT, AXIS>(X, W_b, B_packed, v, Y, M, d_out, d_in, y_dtype, v_stride, g_shift, workspace, sp, stream)
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
