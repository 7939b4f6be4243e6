// What the forms of the hidden update share: recur.hip (launches of their own) and step_few.hip (inside the step's launch).
#pragma once

#include "device_utils.h"
#include "rnnlm_internal.h"

namespace rnnlm {

__device__ __forceinline__ float sigmoid_f32(float a) {
    // 1/(1+2^(-a log2 e)); the hardware exp2/rcp are accurate to about 1 ulp
    return __frcp_rn(1.0f + fast_exp2(-a * kLog2e));
}

// MFMA 32x32x16 operand layout (lane l, g = l / 32):
//   A: 8 consecutive k of row (l % 32), starting at 8 g;   B: same for column (l % 32);
//   D: acc[i] is row 8 (i / 4) + 4 g + i % 4, column l % 32.
__device__ __forceinline__ f32x16 mma(const u32x4 &a, const u32x4 &b, const f32x16 &c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// The first TERMS bf16 terms of eight floats (each the rounded rest of those before it).
template <int TERMS>
__device__ __forceinline__ void bf16_terms(const float (&x)[8], u32x4 (&t)[TERMS]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float a = x[2 * i], b = x[2 * i + 1];
#pragma unroll
        for (int k = 0; k < TERMS; ++k) {
            t[k][i] = pack_bf16x2(a, b);
            a -= __uint_as_float(t[k][i] << 16);
            b -= __uint_as_float(t[k][i] & 0xFFFF0000u);
        }
    }
}

// Embedding row piece: four values of the weights' type.
__device__ __forceinline__ f32x4 load4(const bf16_t *p) {
    const uint2 v = *reinterpret_cast<const uint2 *>(p);
    return f32x4{__uint_as_float(v.x << 16), __uint_as_float(v.x & 0xFFFF0000u), __uint_as_float(v.y << 16),
                 __uint_as_float(v.y & 0xFFFF0000u)};
}
__device__ __forceinline__ f32x4 load4(const float *p) { return *reinterpret_cast<const f32x4 *>(p); }

}  // namespace rnnlm
