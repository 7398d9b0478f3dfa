// The table entry of pass two computed on demand (HIP translation units only).
#pragma once

#include "common.h"

namespace dcpq {

// Double-precision squared distance between a query sub-vector and a centroid row (Eq. 1), rounded to fp32
// once: the value a full table holds.
__device__ inline float entry_on_demand(const float *__restrict__ yj, const float *__restrict__ cen, int dsub, bool vec4)
{
    double dj = 0.0;
    if (vec4) {
#pragma unroll 4
        for (int tt = 0; tt < dsub; tt += 4) {
            const float4 cv = *reinterpret_cast<const float4 *>(cen + tt);
            const float4 yv = *reinterpret_cast<const float4 *>(yj + tt);
            const double d0 = static_cast<double>(yv.x) - static_cast<double>(cv.x);
            const double d1 = static_cast<double>(yv.y) - static_cast<double>(cv.y);
            const double d2 = static_cast<double>(yv.z) - static_cast<double>(cv.z);
            const double d3 = static_cast<double>(yv.w) - static_cast<double>(cv.w);
            dj = fma(d0, d0, dj); dj = fma(d1, d1, dj); dj = fma(d2, d2, dj); dj = fma(d3, d3, dj);
        }
    } else {
        for (int tt = 0; tt < dsub; ++tt) {
            const double df = static_cast<double>(yj[tt]) - static_cast<double>(cen[tt]);
            dj = fma(df, df, dj);
        }
    }
    return static_cast<float>(dj);
}

}  // namespace dcpq
