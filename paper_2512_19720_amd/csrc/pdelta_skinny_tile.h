// Pieces shared by the decode kernels: the 16x16x32 matrix instruction and the operands of the sign part.
#pragma once

#include "pdelta_device.h"

namespace pdelta {

template <int DT>
__device__ __forceinline__ float4v mfma16(uint4v a, uint4v b, float4v c) {
    if constexpr (DT == kBF16)
        return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a),
                                                       __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    else
        return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8, a),
                                                      __builtin_bit_cast(half8, b), c, 0, 0, 0);
}

// Eight sign bits (bit e <-> element e, 1 = +1) to eight +-1.0 values of dtype DT.
template <int DT>
__device__ __forceinline__ uint4v expand_signs(uint32_t byte) {
    constexpr uint32_t one2 = DT == kBF16 ? 0x3F803F80u : 0x3C003C00u;
    const uint32_t neg = ~byte;
    uint4v r;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const uint32_t t = neg >> (2 * p);
        r[p] = one2 | ((t & 1u) << 15) | ((t & 2u) << 30);
    }
    return r;
}

// Column mode: the sign-part operand is fp16(X * v_col), whatever the dtype of X.
template <int XDT>
__device__ __forceinline__ uint4v scale_x(uint4v x, uint4v v) {
    uint4v r;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        if constexpr (XDT == kF16) {
            const uint32_t xp = x[p], vp = v[p];
            r[p] = as_u32(as_half2(xp) * as_half2(vp));                        // v_pk_mul_f16
        } else {
            // (exact products, one rounding to nearest even; two halves at a time)
            typedef float float2v __attribute__((ext_vector_type(2)));
            const uint32_t xp = x[p], vp = v[p];
            const half2v vh = as_half2(vp);
            const float2v prod = {__builtin_bit_cast(float, xp << 16) * (float)vh[0], __builtin_bit_cast(float, xp & 0xFFFF0000u) * (float)vh[1]};
            r[p] = as_u32(__builtin_convertvector(prod, half2v));
        }
    }
    return r;
}

// Grouped scales: the sign-part operands are fp16 whatever the dtype of X: A = fp16(X) and
// B = +-v (the exact product of the +-1 pattern and the group's scale).
template <int XDT>
__device__ __forceinline__ uint4v x_as_f16(uint4v x) {
    if constexpr (XDT == kF16) return x;
    else return scale_x<XDT>(x, (uint4v){0x3C003C00u, 0x3C003C00u, 0x3C003C00u, 0x3C003C00u});
}
__device__ __forceinline__ uint4v signs_times_scale(uint4v pm, uint32_t v_half) {
    const uint32_t vv = v_half | (v_half << 16);
    uint4v r;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const uint32_t sp = pm[p];
        r[p] = as_u32(as_half2(sp) * as_half2(vv));                              // v_pk_mul_f16, exact
    }
    return r;
}

}  // namespace pdelta
