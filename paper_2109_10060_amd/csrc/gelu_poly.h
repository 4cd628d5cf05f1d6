// The short evaluation of GELU behind gelu_bf16x4, free of device types so that the host can check it value by value.
#pragma once

#include <math.h>

#ifdef __HIP__
#define GELU_FN __host__ __device__ __forceinline__
#else
#define GELU_FN inline
#endif

// For |x| <= GELU_LIMIT an odd polynomial (minimax fit of erf(x / sqrt 2) in x^2) gives GELU to within 1.52e-7 |x|, roundings
// included; with the error of gelu_erf, 1.22e-7 |x| on the device, that is inside GELU_SLACK |x|.  (Both are the largest of all
// fp32 values; on the device gelu_bf16x4 and gelu_erf then round to the same bf16 for every one of them.)
constexpr float GELU_LIMIT = 2.5f, GELU_SLACK = 4e-7f;

GELU_FN float gelu_poly(float x) {
    const float u = x * x;
    float p = 1.1145440126369976e-09f;
    p = fmaf(p, u, -5.0059668410540326e-08f);
    p = fmaf(p, u, 1.1413138736315886e-06f);
    p = fmaf(p, u, -1.818383861973416e-05f);
    p = fmaf(p, u, 0.0002292463177582249f);
    p = fmaf(p, u, -0.002372429706156254f);
    p = fmaf(p, u, 0.019945446401834488f);
    p = fmaf(p, u, -0.13298019766807556f);
    p = fmaf(p, u, 0.7978845238685608f);
    const float h = 0.5f * x;
    return fmaf(h, x * p, h);
}
