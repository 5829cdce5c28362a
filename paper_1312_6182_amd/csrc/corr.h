// What the correlation kernels share: the threshold of a correlation and the split
// of FP32 values for the bfloat16 matrix cores.
#pragma once

#include <hip/hip_runtime.h>

namespace gpspca {

// Threshold of one correlation (Table 1).  Returns true when the entry is in
// the support; s is the thresholded value and fv its objective term.
__device__ __forceinline__ bool threshold(bool l0, double mu, double gamma, float y, float& s,
                                          double& fv) {
    const double yd = (double)y;
    if (l0) {
        const double my = mu * yd;
        const double q = my * my - gamma;
        if (q > 0.0) { s = (float)my; fv = q; return true; }
    } else {
        const double t = mu * fabs(yd) - gamma;
        if (t > 0.0) { s = (float)(yd > 0.0 ? t : -t); fv = t * t; return true; }
    }
    s = 0.f;
    fv = 0.0;
    return false;
}

typedef float f4x __attribute__((ext_vector_type(4)));
typedef __bf16 bf8x __attribute__((ext_vector_type(8)));

// v = v1 + v2 + v3, each part bfloat16 (8 significant bits of the 24), exactly.
__device__ __forceinline__ void split3_bf16(const f4x& q0, const f4x& q1, bf8x& v1, bf8x& v2,
                                            bf8x& v3) {
    float r[8];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        r[e] = q0[e];
        r[4 + e] = q1[e];
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        v1[e] = (__bf16)r[e];
        r[e] -= (float)v1[e];
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        v2[e] = (__bf16)r[e];
        r[e] -= (float)v2[e];
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) v3[e] = (__bf16)r[e];
}

}  // namespace gpspca
