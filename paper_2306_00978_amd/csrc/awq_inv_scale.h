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
