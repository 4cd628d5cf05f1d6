// GELU with the exact erf, and its bf16 rounding without the cost of erff.
#pragma once

#include "common.h"
#include "gelu_poly.h"

__device__ __forceinline__ float gelu_erf(float x) { return 0.5f * x * (1.0f + erff(x * 0.70710678118654752f)); }

// Four values -> packed bf16, bit for bit f2bf2 of gelu_erf.  erff costs about 25 vector instructions and two branches a
// value; between two and three of four rounded results are decided by far less precision.  gelu_poly is within GELU_SLACK |x|
// of gelu_erf up to |x| = 2.5; where the bounds of that interval round to the same bf16, so does gelu_erf.  A group of lanes
// with a value outside, or too close to a rounding boundary (about one value in 3000), takes gelu_erf itself.
__device__ __forceinline__ uint2 gelu_bf16x4(float x0, float x1, float x2, float x3) {
    const float x[4] = {x0, x1, x2, x3};
    float lo[4], hi[4], top = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const float r = gelu_poly(x[i]), a = fabsf(x[i]);
        lo[i] = fmaf(-GELU_SLACK, a, r);
        hi[i] = fmaf(GELU_SLACK, a, r);
        top = fmaxf(top, a);
    }
    uint2 q = make_uint2(f2bf2(lo[0], lo[1]), f2bf2(lo[2], lo[3]));
    const uint32_t d = (q.x ^ f2bf2(hi[0], hi[1])) | (q.y ^ f2bf2(hi[2], hi[3]));
    if (d != 0 || !(top <= GELU_LIMIT)) {
        q.x = f2bf2(gelu_erf(x0), gelu_erf(x1));
        q.y = f2bf2(gelu_erf(x2), gelu_erf(x3));
    }
    return q;
}
