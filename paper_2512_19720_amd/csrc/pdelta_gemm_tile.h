// Pieces shared by the prefill kernels: conversion of staged operands and the epilogue of a wave tile.
#pragma once

#include "pdelta_device.h"

namespace pdelta {

constexpr int kGemmBN = 128, kGemmBK = 64;
constexpr int kGemmLDK = kGemmBK + 8;   // padded LDS row in halves (144 bytes)
constexpr int kXcds = 8;

__device__ __forceinline__ uint32_t bf16pair_to_f16pair(uint32_t d) {
    const float lo = __builtin_bit_cast(float, d << 16);
    const float hi = __builtin_bit_cast(float, d & 0xFFFF0000u);
    return as_u32(__builtin_bit_cast(half2v, __builtin_amdgcn_cvt_pkrtz(lo, hi)));
}

template <int XDT>
__device__ __forceinline__ uint4v to_f16x8(uint4v a) {
    if constexpr (XDT == kBF16) {
        uint4v r;
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const uint32_t ap = a[p];
            r[p] = bf16pair_to_f16pair(ap);
        }
        return r;
    } else {
        return a;
    }
}

// Eight fp16 weights and eight "negate" bits (bit e set: element e gets -|v|, clear: +|v|) with
// the packed magnitudes |v| of elements 2p (low half) and 2p+1 (high half) in vabs[p].
// Row mode: |v| is one value per row and the sign of v is folded into the bits by the caller.
__device__ __forceinline__ uint4v add_signed_scale(uint4v w, uint32_t negbits, uint4v vabs) {
    uint4v r;
    negbits &= 0xFFu;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        // bit 2p -> position 15, bit 2p+1 -> position 31; everything else is masked by the insert
        const uint32_t spread = (negbits << (30 - 2 * p)) | (negbits << (15 - 2 * p));
        const uint32_t va = vabs[p], wp = w[p];
        const uint32_t sv = (spread & 0x80008000u) | (va & 0x7FFF7FFFu);        // v_bfi_b32
        r[p] = as_u32(as_half2(wp) + as_half2(sv));                              // v_pk_add_f16
    }
    return r;
}

// Epilogue of the 64 x 64 wave tile for 16-bit outputs: the accumulators go through a wave-private
// LDS region (32 rows x 64 columns at a time, rows padded to 144 bytes) and leave as 16-byte
// stores, eight lanes per 128-byte line of Y, instead of 64 two-byte store instructions per
// accumulator tile (measured 2-3 % of the run time).  `region` holds 32 * kGemmLDK halves of this wave.
// Returns false (nothing stored) when the tile is not fully inside Y or rows of Y are not
// 16-byte aligned; the caller then stores element by element.
template <int FM>
__device__ __forceinline__ bool store_tile_16bit(const float16v (&acc)[FM][2], uint16_t* region, void* Y,
                                                 int y_dtype, int tok0, int o0, int M, int d_out, int lane)
{
    if (y_dtype == kF32 || (d_out & 7) != 0 || o0 + 64 > d_out || tok0 + FM * 32 > M) return false;   // wave-uniform
    uint16_t* Yh = (uint16_t*)Y;
#pragma unroll
    for (int f = 0; f < FM; ++f) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int row = (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3), col = h * 32 + (lane & 31);
                const float val = acc[f][h][r];
                region[row * kGemmLDK + col] =
                    (uint16_t)(y_dtype == kBF16 ? f32_to_bf16_bits(val) : f32_to_f16_bits(val));
            }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
#pragma unroll
        for (int it = 0; it < 4; ++it) {
            const int row = it * 8 + (lane >> 3), chunk = lane & 7;
            const uint4v vals = *(const uint4v*)(region + row * kGemmLDK + chunk * 8);
            *(uint4v*)(Yh + (int64_t)(tok0 + f * 32 + row) * d_out + o0 + chunk * 8) = vals;
        }
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
    return true;
}

// The wave tile's outputs, 16-bit outputs inside Y through `region`, the others element by element.
// 32x32 accumulator: element r of lane l is row (r/4)*8 + (l/32)*4 + r%4, column l%32.
template <int FM>
__device__ __forceinline__ void store_wave_tile(const float16v (&acc)[FM][2], uint16_t* region, void* Y, int y_dtype,
                                                int tok0, int o0, int M, int d_out, int lane)
{
    if (store_tile_16bit<FM>(acc, region, Y, y_dtype, tok0, o0, M, d_out, lane)) return;
#pragma unroll
    for (int f = 0; f < FM; ++f)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int o = o0 + h * 32 + (lane & 31);
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int tok = tok0 + f * 32 + (r >> 2) * 8 + (lane >> 5) * 4 + (r & 3);
                if (tok < M && o < d_out) {
                    const int64_t yi = (int64_t)tok * d_out + o;
                    const float val = acc[f][h][r];
                    if (y_dtype == kF32) store_y<kF32>(Y, yi, val);
                    else if (y_dtype == kBF16) store_y<kBF16>(Y, yi, val);
                    else store_y<kF16>(Y, yi, val);
                }
            }
        }
}

}  // namespace pdelta
