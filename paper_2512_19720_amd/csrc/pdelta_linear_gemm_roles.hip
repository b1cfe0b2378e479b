// Prefill-shaped delta linear layer on few tiles, d_in a multiple of 128: the arithmetic of pdelta_linear_gemm.hip (W_hat =
// fp16(W_b +- v), X as fp16, fp32 sums in the order of d_in) on tiles of 64 tokens x 64 output rows with the work of a
// workgroup split by role.
//
// 251 tokens on 4096 outputs are 256 such tiles, one per CU, and the sums of an output run in order: the time is that of 4096
// inputs, one after another, on four waves that multiply.  In linear_gemm_small_kernel the same four waves also load,
// convert and stage, and a step of 64 inputs takes 0.4 us, several times its MFMAs and LDS traffic.  Here four waves only
// read fragments and multiply, eight others load W_b into registers three pairs of steps ahead, convert and stage it
// (bf16: X too; fp16 X comes by direct loads into LDS from the multiplying waves), and there is one barrier for 128 inputs.
// What is left is the chain from barrier to barrier: counters of 251 tokens, 4096 x 4096 fp16 col show 1440 cycles per 128
// inputs, of which the LDS is busy 27 %, the vector ALUs 23 %, the matrix cores 18 %, and without any load 17 us of 25 remain.
// 52 MB are fetched, X once per XCD.  An L2 touch ahead of the loads, whole 2 KB of a row at a time or
// line by line, costs 1-2 us; a fourth pair in registers changes nothing.
//
// Calls in a row in a graph, weights changing, 251 tokens, 4096 x 4096, us, linear_gemm_small_kernel -> this one: fp16 row 28.5
// -> 24.5, col 30.5 -> 26.2, blockwise 31.2 -> 26.8, bf16 row 32.7 -> 25.5, col 35.6 -> 28.1; 128 tokens fp16 row 28.8 -> 24.8;
// 100 tokens, 1024 x 1024 fp16 9.4 -> 7.5.  Where the inputs still lie in the memory-side cache (six sets of them, calls one by
// one), 251 tokens fp16 col 28.8 -> 21.4.
#include <type_traits>

#include "pdelta_gemm_tile.h"
#include "pdelta_host.h"
#include "pdelta_lds_load.h"

namespace pdelta {

constexpr int kRolePairK = 128;                       // inputs between two barriers
constexpr int kRoleHalf = 64 * 128, kRoleTile = 2 * kRoleHalf;       // bytes of 64 rows x 64 (128) inputs
constexpr int kRoleThreads = 12 * 64;
constexpr int kRoleXStages = 4, kRoleRing = 3;        // pairs of X in LDS (fp16); pairs in the stagers' registers

// What a stager holds of one pair: 16 bytes of W_b (bf16: and of X) of each half, the signs and scales that go with them.
template <int XDT, int AXIS>
struct RoleRegs {
    uint4v w[2], x[XDT == kBF16 ? 2 : 1], v[AXIS == 1 ? 2 : 1];
    uint32_t sb[2], vg[2];
};

// Whether whole output-row tiles go to the XCDs in turn: while no XCD gets more tiles than its 32 CUs, of which each holds one
// workgroup.  Above that the busiest XCD takes twice as long (1224 tokens x 628 x 256 fp16 col 9.5 us, 7.2 with consecutive tiles; 332
// x 2634 x 768 bf16 10.1 and 7.5); below, fp16 calls are 1-4 % faster (94 x 1792 x 2560 row 12.6 and 13.1) and bf16 even.
__host__ __device__ inline bool role_columns(int m_tiles, int n_tiles)
{
    return (int64_t)m_tiles * ((n_tiles + kXcds - 1) / kXcds) <= 256 / kXcds;
}

template <int XDT, int AXIS>
__global__ void __launch_bounds__(kRoleThreads, 3)
linear_gemm_roles_kernel(const uint16_t* __restrict__ X, const uint16_t* __restrict__ W_b, const uint32_t* __restrict__ B_packed,
                         const uint16_t* __restrict__ v, void* __restrict__ Y, int M, int d_out, int d_in, int y_dtype,
                         int m_tiles, int n_tiles, int v_stride, int g_shift)
{
    constexpr bool XDMA = XDT == kF16;                // X needs no conversion: direct loads, by the multiplying waves
    constexpr int XST = XDMA ? kRoleXStages : 2, WBUF = XST * kRoleTile;
    extern __shared__ __attribute__((aligned(16))) unsigned char role_lds[];     // [XST] tiles of X, [2] of W_hat

    // The XCDs take output-row tiles in turn, each with all its token tiles, or, where one would get more tiles than it has CUs,
    // consecutive tiles, at most its eighth (see role_columns).
    const int xcd = blockIdx.x % kXcds, local = blockIdx.x / kXcds, per_xcd = gridDim.x / kXcds;
    const bool columns = role_columns(m_tiles, n_tiles);
    const int tile = columns ? (local / m_tiles * kXcds + xcd) * m_tiles + local % m_tiles : xcd * per_xcd + local;
    if (tile >= m_tiles * n_tiles) return;            // whole workgroup
    const int tile_n = tile / m_tiles, tile_m = tile % m_tiles;
    const int n0 = tile_n * 64, m0 = tile_m * 64;
    const int K = d_in, n_pairs = K / kRolePairK;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);

    const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)role_lds);

    if (wave >= 4) {
        // ---- stagers: wave h of 8 has rows 8 h .. + 7, a lane 16 bytes of each half of its row ----
        const int h = wave - 4, row = h * 8 + (lane >> 3), p = lane & 7;
        const int wr = min(n0 + row, d_out - 1), xr = min(m0 + row, M - 1);
        const char* wbase = (const char*)(W_b + (int64_t)n0 * K);
        const char* xbase = (const char*)(X + (int64_t)m0 * K);
        const char* sbase = (const char*)B_packed + (int64_t)n0 * (K >> 3);
        const uint32_t woff = (uint32_t)(wr - n0) * (uint32_t)K * 2u + p * 16u, xoff = (uint32_t)(xr - m0) * (uint32_t)K * 2u + p * 16u;
        const uint32_t soff = (uint32_t)(wr - n0) * (uint32_t)(K >> 3) + p;
        const uint32_t vrow = AXIS == 0 ? (uint32_t)v[wr] * 0x10001u : 0u;
        const uint16_t* vg = AXIS == 2 ? v + (int64_t)wr * v_stride : v;
        unsigned char* const to = role_lds + row * 128 + ((p ^ ((row >> 1) & 7)) * 16);
        auto load = [&](RoleRegs<XDT, AXIS>& R, int pair) {
            const int kb = pair * kRolePairK;
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                R.w[q] = *(const uint4v*)(wbase + (int64_t)kb * 2 + q * 128 + woff);
                R.sb[q] = (uint32_t) * (const uint8_t*)(sbase + (kb >> 3) + q * 8 + soff);
                if constexpr (!XDMA) R.x[q] = *(const uint4v*)(xbase + (int64_t)kb * 2 + q * 128 + xoff);
                if constexpr (AXIS == 1) R.v[q] = *(const uint4v*)(v + kb + q * 64 + p * 8);
                if constexpr (AXIS == 2) R.vg[q] = vg[(kb + q * 64 + p * 8) >> g_shift];
            }
        };
        auto convert = [&](const RoleRegs<XDT, AXIS>& R, int buf) {
#pragma unroll
            for (int q = 0; q < 2; ++q) {
                const uint32_t neg = ~R.sb[q] & 0xFFu;
                uint32_t y = neg | (neg << 15);       // bit 2e + 1 at 2e + 16
                asm("" : "+v"(y));                    // (else y and its shifts become full multiplications)
                const uint32_t vv = AXIS == 2 ? R.vg[q] | (R.vg[q] << 16) : vrow;
                const uint4v w16 = to_f16x8<XDT>(R.w[q]);
                uint4v r;
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const uint32_t vp = AXIS == 1 ? R.v[q][e] : vv, wp = w16[e];
                    const uint32_t sv = ((y << (15 - 2 * e)) & 0x80008000u) ^ vp;     // -v where the bit is set
                    r[e] = as_u32(as_half2(wp) + as_half2(sv));
                }
                *(uint4v*)(to + WBUF + buf * kRoleTile + q * kRoleHalf) = r;
                if constexpr (!XDMA) *(uint4v*)(to + buf * kRoleTile + q * kRoleHalf) = to_f16x8<kBF16>(R.x[q]);
            }
        };
        RoleRegs<XDT, AXIS> R[kRoleRing];
#pragma unroll
        for (int d = 0; d < kRoleRing; ++d) load(R[d], min(d, n_pairs - 1));
        convert(R[0], 0);
        load(R[0], min(kRoleRing, n_pairs - 1));
        lds_barrier();
        // While pair i is multiplied: pair i + 1 to LDS, pair i + 1 + kRoleRing asked for (clamped at the end).  No branch
        // in the loop: at the join after one the compiler waits for every load in flight.
        auto period = [&](int i, RoleRegs<XDT, AXIS>& next) {
            convert(next, (i + 1) & 1);
            load(next, min(i + 1 + kRoleRing, n_pairs - 1));
            lds_barrier();
        };
        int i = 0;
        for (; i + kRoleRing < n_pairs; i += kRoleRing) {
#pragma unroll
            for (int d = 0; d < kRoleRing; ++d) period(i + d, R[(d + 1) % kRoleRing]);
        }
#pragma unroll
        for (int d = 0; d < kRoleRing; ++d) {
            if (i + d + 1 < n_pairs) convert(R[(d + 1) % kRoleRing], (i + d + 1) & 1);
            if (i + d < n_pairs) lds_barrier();
        }
        return;
    }

    // ---- multipliers: wave (wm, wn) has 32 tokens x 32 output rows ----
    const int wm = wave >> 1, wn = wave & 1;
    const char* xbase = (const char*)(X + (int64_t)m0 * K);
    uint32_t xoff[4];                                 // load q: rows 8 (4 (wave & 1) + q) .. + 7 of half wave >> 1
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const int rg = (wave & 1) * 4 + q;
        xoff[q] = (uint32_t)(min(m0 + rg * 8 + (lane >> 3), M - 1) - m0) * (uint32_t)K * 2u + (wave >> 1) * 128u +
                  (uint32_t)((lane & 7) ^ ((rg & 1) * 4 + (lane >> 4))) * 16u;
    }
    auto request = [&](int pair) {
        const uint32_t at = __builtin_amdgcn_readfirstlane(lds0 + (pair % XST) * kRoleTile + (wave >> 1) * kRoleHalf + (wave & 1) * 4096);
#pragma unroll
        for (int q = 0; q < 4; ++q) load_lds_16(at + q * 1024, xoff[q], xbase + (int64_t)pair * (kRolePairK * 2));
    };
    auto wait_for = [&](int later) {                  // all but the loads of that many pairs
        if (later >= 2) wait_loads<8>();
        else if (later == 1) wait_loads<4>();
        else wait_loads<0>();
    };
    float16v acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
    const uint32_t frag = (uint32_t)((lane & 31) * 128 + (((lane >> 5) ^ ((lane >> 1) & 7)) * 16));     // of 16 inputs ks: ^ 32 ks
    if constexpr (XDMA) {
#pragma unroll
        for (int d = 0; d < XST - 1; ++d)
            if (d < n_pairs) request(d);
        wait_for(min(n_pairs, XST - 1) - 1);
    }
    lds_barrier();
    for (int i = 0; i < n_pairs; ++i) {
        const unsigned char* xa = role_lds + (XDMA ? i % XST : i & 1) * kRoleTile + wm * 4096;
        const unsigned char* wa = role_lds + WBUF + (i & 1) * kRoleTile + wn * 4096;
        if constexpr (XDMA) if (i + XST - 1 < n_pairs) request(i + XST - 1);      // (into the stage of pair i - 1)
        half8 a[8], b[8];                             // four fragments ahead of the products
        auto frags = [&](int ks) {
            a[ks] = *(const half8*)(xa + (ks >> 2) * kRoleHalf + (frag ^ ((ks & 3) * 32)));
            b[ks] = *(const half8*)(wa + (ks >> 2) * kRoleHalf + (frag ^ ((ks & 3) * 32)));
        };
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) frags(ks);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) {
            if (ks + 4 < 8) frags(ks + 4);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(a[ks], b[ks], acc, 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (XDMA) if (i + 1 < n_pairs) wait_for(min(n_pairs - 2 - i, XST - 2));
        lds_barrier();
    }

    const int o = n0 + wn * 32 + (lane & 31);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const int tok = m0 + wm * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
        if (tok < M && o < d_out) {
            const int64_t yi = (int64_t)tok * d_out + o;
            if (y_dtype == kF32) store_y<kF32>(Y, yi, acc[r]);
            else if (y_dtype == kBF16) store_y<kBF16>(Y, yi, acc[r]);
            else store_y<kF16>(Y, yi, acc[r]);
        }
    }
}

template <int XDT, int AXIS>
static int launch_roles(const void* X, const void* W_b, const uint32_t* B_packed, const uint16_t* v, void* Y, int64_t M,
                        int64_t d_out, int64_t d_in, int y_dtype, int v_stride, int g_shift, hipStream_t stream)
{
    constexpr int lds = ((XDT == kF16 ? kRoleXStages : 2) + 2) * kRoleTile;      // 98,304 (fp16) or 65,536 bytes
    auto kernel = linear_gemm_roles_kernel<XDT, AXIS>;
    static unsigned lds_opted_in = 0;                 // per template instance: one kernel
    if (opt_in_dynamic_lds((const void*)kernel, lds, &lds_opted_in) != 0) return -1;
    const int m_tiles = (int)((M + 63) / 64), n_tiles = (int)((d_out + 63) / 64);
    const int per_xcd = role_columns(m_tiles, n_tiles) ? (n_tiles + kXcds - 1) / kXcds * m_tiles : (m_tiles * n_tiles + kXcds - 1) / kXcds;
    hipLaunchKernelGGL(kernel, dim3((unsigned)(per_xcd * kXcds)), dim3(kRoleThreads), lds, stream, (const uint16_t*)X,
                       (const uint16_t*)W_b, B_packed, v, Y, (int)M, (int)d_out, (int)d_in, y_dtype, m_tiles, n_tiles, v_stride, g_shift);
    return hipGetLastError() == hipSuccess ? 0 : -1;
}

int launch_linear_gemm_roles(int x_dtype, int y_dtype, int axis, const void* X, const void* W_b, const uint32_t* B_packed,
                             const uint16_t* v, void* Y, int64_t M, int64_t d_out, int64_t d_in, int v_stride, int g_shift,
                             hipStream_t stream)
{
#define PDELTA_GO(XDT, AXIS) return launch_roles<XDT, AXIS>(X, W_b, B_packed, v, Y, M, d_out, d_in, y_dtype, v_stride, g_shift, stream)
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
