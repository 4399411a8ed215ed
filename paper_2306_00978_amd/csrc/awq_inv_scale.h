// Eight activations divided by their channels' scales (Eq. 4): fp32 division, one rounding to fp16.
#pragma once

#include "awq_common.h"

__device__ __forceinline__ uint4 inv_scaled(const uint4 &raw, const float4 &a, const float4 &b)
{
    const half_t *h = reinterpret_cast<const half_t *>(&raw);
    const float sv[8] = {a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
    uint4 out;
    half_t *o = reinterpret_cast<half_t *>(&out);
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = (half_t)((float)h[e] / sv[e]);
    return out;
}

// The same with the reciprocals y = 1 / s (correctly rounded) at hand: the quotient from one multiplication and two fused
// multiply-adds is the correctly rounded one for every half x and every s between 2^-60 and 2^60 (proved exhaustively over
// the significands by tests/reciprocal_quotient_check.c); the fix-up is the division's own, for zeros, infinities and NaN.
// 22 cycles an element where the compiler's division takes 55.
__device__ __forceinline__ float quotient_by(float x, float s, float y)
{
    const float q0 = x * y;
    const float e = __builtin_fmaf(-q0, s, x);
    return __builtin_amdgcn_div_fixupf(__builtin_fmaf(e, y, q0), s, x);
}

__device__ __forceinline__ uint4 inv_scaled_by(const uint4 &raw, const float (&s)[8], const float (&y)[8])
{
    const half_t *h = reinterpret_cast<const half_t *>(&raw);
    uint4 out;
    half_t *o = reinterpret_cast<half_t *>(&out);
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] = (half_t)quotient_by((float)h[e], s[e], y[e]);
    return out;
}
