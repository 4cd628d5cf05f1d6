// The short evaluation of GELU behind gelu_bf16x4, free of device types so that the host can check it value by value.
#pragma once

#include <math.h>

#ifdef __HIP__
#define GELU_FN __host__ __device__ __forceinline__
#else
#define GELU_FN inline
#endif

// For |x| <= GELU_LIMIT gelu(x) = x / 2 + x^2 P(x^2): the second half is even.  P is a minimax fit in x^2 - GELU_MIDDLE, about the middle of the
// range, where its terms do not cancel: within 1.04e-7 |x| of GELU with every rounding (largest of all fp32 values; root mean square 2.0e-8), where
// gelu_erf is within 1.22e-7 |x| on the device.  In x^2 itself nine terms up to 2.5 were good to 1.52e-7 |x|.
// GELU_SLACK |x|: how far two fp32 evaluations may lie apart, this one and gelu_erf, roundings included.
constexpr float GELU_LIMIT = 3.5f, GELU_SLACK = 4e-7f;

constexpr int GELU_TERMS = 12;
constexpr float GELU_MIDDLE = 6.5f;
constexpr float GELU_P[GELU_TERMS] = {0.19400054216384888f, -0.013733221217989922f, 0.0012871280778199434f, -0.00011543738946784288f,
                                      9.342209523310885e-06f, -6.737686817359645e-07f, 4.3392351045667965e-08f, -2.5126627445359873e-09f,
                                      1.3000769905069376e-10f, -6.042295136454712e-12f, 3.1192103479120437e-13f, -1.460037636852405e-14f};

GELU_FN float gelu_poly(float x) {
    const float u = x * x, s = fmaf(x, x, -GELU_MIDDLE);
    float p = GELU_P[GELU_TERMS - 1];
#pragma GCC unroll 16
    for (int i = GELU_TERMS - 2; i >= 0; --i) p = fmaf(p, s, GELU_P[i]);
    return fmaf(u, p, 0.5f * x);
}
