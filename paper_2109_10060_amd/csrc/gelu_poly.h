// The short evaluation of GELU behind gelu_bf16x4, free of device types so that the host can check it value by value.
#pragma once

#include <math.h>

#ifdef __HIP__
#define GELU_FN __host__ __device__ __forceinline__
#else
#define GELU_FN inline
#endif

// For |x| <= GELU_LIMIT gelu(x) = x / 2 + x^2 P(x^2): the second half is even.  P is a minimax fit in x^2 - GELU_MIDDLE, about the middle of the
// range, where its terms do not cancel.  Error of |x|, every rounding in it, against double: 1.04e-7 at most over all fp32 values, where gelu_erf is
// within 1.22e-7 on the device.  By ranges of x, root mean square over evenly spaced values, here / by erff (the host's), and bf16 results of a million that are
// not the nearest:
//   -3.5..-3   2.2e-8 / 0.9e-8   6600 / 2900      -0.5..0.5  1.4e-8 / 2.0e-8   7 / 6
//   -3..-2.5   1.7e-8 / 0.9e-8    940 / 510        0.5..1.5  2.6e-8 / 3.1e-8   9 / 10
//   -2.5..-1.5 1.7e-8 / 1.0e-8    130 / 80         1.5..2.5  3.0e-8 / 3.4e-8   9 / 7
//   -1.5..-0.5 1.6e-8 / 1.2e-8     19 / 11         2.5..3.5  3.0e-8 / 3.3e-8   8 / 7
// So it is the better one where GELU is large, and by up to two and a half times the worse one on the negative half, where x / 2 and the even half cancel and
// the result is small beside |x|.  Over normally distributed values (not relative to them), here / by erff: deviation 0.3 4.9e-9 / 6.4e-9, 0.8 1.79e-8 /
// 1.91e-8, 1.2 2.88e-8 / 2.93e-8, 2 4.91e-8 / 4.85e-8.
constexpr float GELU_LIMIT = 3.5f;

constexpr int GELU_TERMS = 12;
constexpr float GELU_MIDDLE = 6.5f;
constexpr float GELU_P[GELU_TERMS] = {0.19400054216384888f, -0.013733221217989922f, 0.0012871280778199434f, -0.00011543738946784288f,
                                      9.342209523310885e-06f, -6.737686817359645e-07f, 4.3392351045667965e-08f, -2.5126627445359873e-09f,
                                      1.3000769905069376e-10f, -6.042295136454712e-12f, 3.1192103479120437e-13f, -1.460037636852405e-14f};

// The steps of a value, 0 .. GELU_TERMS; the last one leaves the result in p.  HALF: of x / 2 in place of x, an instruction less.  With the terms' powers of
// four in the constants every sum is the other one's times a power of two, and so the result is the same bits (|x| < 2^-125: to the last of a subnormal).
constexpr float gelu_term(int i, bool half) { return half ? GELU_P[i] * (float)(4u << 2 * i) : GELU_P[i]; }
template <bool HALF>
GELU_FN void gelu_step(int l, float x, float& u, float& s, float& p) {
    if (l == 0) {
        u = x * x;
        s = fmaf(x, x, HALF ? -GELU_MIDDLE / 4 : -GELU_MIDDLE);
        p = gelu_term(GELU_TERMS - 1, HALF);
    } else if (l < GELU_TERMS) p = fmaf(p, s, gelu_term(GELU_TERMS - 1 - l, HALF));
    else p = fmaf(u, p, HALF ? x : 0.5f * x);
}

GELU_FN float gelu_poly(float x) {
    float u, s, p;
#pragma GCC unroll 16
    for (int l = 0; l <= GELU_TERMS; ++l) gelu_step<false>(l, x, u, s, p);
    return p;
}
