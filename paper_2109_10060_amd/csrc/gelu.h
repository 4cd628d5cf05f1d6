// GELU with the exact erf: by erff, and for bf16 results by one polynomial of the same precision.
#pragma once

#include "common.h"
#include "gelu_poly.h"

__device__ __forceinline__ float gelu_erf(float x) { return 0.5f * x * (1.0f + erff(x * 0.70710678118654752f)); }

// A group of four values of which one or more lie outside gelu_poly's range: those by gelu_erf in place of q's, one erff after the other (a loop: the code
// of a kernel holds many such groups).  HALF: the x are halves of the values.
template <bool HALF = false>
__device__ __forceinline__ uint2 gelu_bf16x4_far(uint2 q, float x0, float x1, float x2, float x3) {
    constexpr float LIMIT = HALF ? GELU_LIMIT / 2 : GELU_LIMIT;
    const uint2 far = make_uint2((fabsf(x0) > LIMIT ? 0xffffu : 0u) | (fabsf(x1) > LIMIT ? 0xffff0000u : 0u),
                                 (fabsf(x2) > LIMIT ? 0xffffu : 0u) | (fabsf(x3) > LIMIT ? 0xffff0000u : 0u));
    float y0 = 0.f, y1 = 0.f, y2 = 0.f, y3 = 0.f;
#pragma unroll 1
    for (int i = 0; i < 4; ++i) {
        const float y = gelu_erf(HALF ? 2.f * x0 : x0);
        x0 = x1, x1 = x2, x2 = x3;
        y0 = y1, y1 = y2, y2 = y3, y3 = y;
    }
    return make_uint2((q.x & ~far.x) | (f2bf2(y0, y1) & far.x), (q.y & ~far.y) | (f2bf2(y2, y3) & far.y));
}
__device__ __forceinline__ float gelu_top(float x0, float x1, float x2, float x3) {
    return fmaxf(fmaxf(fabsf(x0), fabsf(x1)), fmaxf(fabsf(x2), fabsf(x3)));      // (a NaN is one by gelu_poly too)
}
__device__ __forceinline__ uint2 gelu_bf16x4_near(float x0, float x1, float x2, float x3) {
    return make_uint2(f2bf2(gelu_poly(x0), gelu_poly(x1)), f2bf2(gelu_poly(x2), gelu_poly(x3)));
}
// Four values -> packed bf16: gelu_poly inside its range, gelu_erf outside, each value for itself.  erff costs about 25 vector instructions
// and two branches a value, gelu_poly 15.  (A shorter polynomial, with a check that its bf16 result is that of erff and erff itself where
// that is open, cost 16 and the check: of the groups of 64 lanes x 4 values one in twelve was done over.)
__device__ __forceinline__ uint2 gelu_bf16x4(float x0, float x1, float x2, float x3) {
    const uint2 q = gelu_bf16x4_near(x0, x1, x2, x3);
    return gelu_top(x0, x1, x2, x3) > GELU_LIMIT ? gelu_bf16x4_far(q, x0, x1, x2, x3) : q;
}
