// Quotients of sizes that a kernel gets as arguments, free of device types so that the host can check them.
#pragma once

#ifdef __HIP__
#define QUOTIENT_FN __host__ __device__ __forceinline__
#else
#define QUOTIENT_FN inline
#endif

// n / d for 0 <= n < 2^31, d > 0; r within two units in the last place of 1 / d.  The first guess is off by n / d 2^-22 and one, the second, of what it leaves, by one.
// (Unsigned, since the first guess and its product may lie beyond 2^31.)  About a dozen vector instructions one behind the other, the compiler's division 30.
QUOTIENT_FN int quotient(int n, int d, float r) {
    unsigned q = (unsigned)((float)n * r);
    auto left = [&]() { return (int)((unsigned)n - q * (unsigned)d); };
    q += (unsigned)(int)((float)left() * r);
    const int m = left();
    return (int)q + (m >= d) - (m < 0);
}
// the same for n < 2^22, where the first guess is off by one at most
QUOTIENT_FN int quotient22(int n, int d, float r) {
    const int q = (int)((float)n * r), m = n - q * d;
    return q + (m >= d) - (m < 0);
}
