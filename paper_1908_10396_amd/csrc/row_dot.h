// The exact score of a point (paper Section 1), as every re-scoring forms it.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace avq {

// <q, x> as an fp32 fma chain in index order. qs: query in LDS.
__device__ __forceinline__ float row_dot_chain(const float *qs, const float *__restrict__ row, int d)
{
    float s = 0.0f;
    if ((d & 3) == 0 && (((uintptr_t)row) & 15) == 0) {
        // five 16-byte loads in flight at a time (the chain itself is serial): a row of 100 floats in five rounds
        const float4 *r4 = (const float4 *)row;
        const int n4 = d / 4;
        int l = 0;
        for (; l + 5 <= n4; l += 5) {
            float4 v[5];
#pragma unroll
            for (int u = 0; u < 5; ++u) v[u] = r4[l + u];
#pragma unroll
            for (int u = 0; u < 5; ++u) {
                s = __fmaf_rn(qs[4 * (l + u) + 0], v[u].x, s);
                s = __fmaf_rn(qs[4 * (l + u) + 1], v[u].y, s);
                s = __fmaf_rn(qs[4 * (l + u) + 2], v[u].z, s);
                s = __fmaf_rn(qs[4 * (l + u) + 3], v[u].w, s);
            }
        }
        for (; l < n4; ++l) {
            const float4 v = r4[l];
            s = __fmaf_rn(qs[4 * l + 0], v.x, s);
            s = __fmaf_rn(qs[4 * l + 1], v.y, s);
            s = __fmaf_rn(qs[4 * l + 2], v.z, s);
            s = __fmaf_rn(qs[4 * l + 3], v.w, s);
        }
    } else {
        for (int l = 0; l < d; ++l) s = __fmaf_rn(qs[l], row[l], s);
    }
    return s;
}

} // namespace avq
