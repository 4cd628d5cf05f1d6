// Depthwise filter rows as band matrices: geometry shared by the kernels that put a depthwise convolution on
// v_mfma_f32_4x4x4_16b_bf16 (one channel per block of the instruction).  A filter row applied to four neighbouring outputs
// is a 4 x (3 stride + N) band matrix times a column of pixels.
#pragma once
#include "common.h"

typedef __attribute__((ext_vector_type(4))) short short4_t;

constexpr uint32_t BAND_OOB = 0x80000000u;

// steps of K = 4 of a filter row, staged pixel quads of a row of strips (4 outputs each)
__host__ __device__ constexpr int band_steps(int n, int stride) { return (3 * stride + n + 3) / 4; }
__host__ __device__ constexpr int band_quads(int strips, int n, int stride) { return (strips - 1) * stride + band_steps(n, stride); }
// bytes of a channel's window: the rows back to back, then up to an odd multiple of 32, so that the 16 lanes of an LDS
// phase (4 channels x 4 strips of 8 bytes) meet every bank once
__host__ __device__ constexpr int band_pitch(int rows, int quads) { return ((rows * quads * 8 + 95) & ~63) - 32; }
// and 16 more behind every 8 channels, for the 8-byte stores of 2..8 channel octets x neighbouring quads
__host__ __device__ constexpr int band_window(int cw, int pitch) { return cw * pitch + cw / 8 * 16; }
// a channel's filter: its rows between zeros, so that row m of a band is a window of it, m strides further left; an odd
// number of dwords per channel against conflicts
__host__ __device__ constexpr int band_lead(int stride) { return 3 * stride; }
__host__ __device__ constexpr int band_row_dwords(int stride) { return stride == 1 ? 8 : 11; }
__host__ __device__ constexpr int band_filter_pitch(int n, int stride) { return (n * band_row_dwords(stride) | 1) * 4; }

#ifdef __HIPCC__
// the bands of the channel whose filter starts at `f`: row m = lane & 3 of filter row i, step t
template <int N, int STRIDE>
__device__ __forceinline__ void band_operand(short4_t (&A)[N][band_steps(N, STRIDE)], const char* f) {
    constexpr int T = band_steps(N, STRIDE);
    const int e = band_lead(STRIDE) - (threadIdx.x & 3) * STRIDE;    // row m starts here
    const uint32_t* p = (const uint32_t*)f + (e >> 1);
#pragma unroll
    for (int i = 0; i < N; ++i) {
        uint32_t v[2 * T];
#pragma unroll
        for (int k = 0; k < 2 * T; ++k) v[k] = p[i * band_row_dwords(STRIDE) + k];
        if constexpr (STRIDE == 1) {
            const uint32_t last = p[i * band_row_dwords(STRIDE) + 2 * T];
#pragma unroll
            for (int k = 0; k < 2 * T; ++k) v[k] = __builtin_amdgcn_alignbit(k + 1 < 2 * T ? v[k + 1] : last, v[k], (e & 1) * 16);
        }
#pragma unroll
        for (int t = 0; t < T; ++t) A[i][t] = __builtin_bit_cast(short4_t, make_uint2(v[2 * t], v[2 * t + 1]));
    }
}

// RO output rows of a strip: every input row (r-th at p + at(r)) is read once and added to the outputs it touches
template <int N, int STRIDE, int RO, typename At>
__device__ __forceinline__ void band_rows_at(f32x4_t (&acc)[RO], const short4_t (&A)[N][band_steps(N, STRIDE)], const char* p, At at) {
    constexpr int T = band_steps(N, STRIDE), ROWS = (RO - 1) * STRIDE + N;
#pragma unroll
    for (int y = 0; y < RO; ++y) acc[y] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int r = 0; r < ROWS; ++r) {
        short4_t B[T];
#pragma unroll
        for (int t = 0; t < T; ++t) B[t] = *(const short4_t*)(p + at(r) + t * 8);
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
            for (int y = 0; y < RO; ++y)
                if (r - y * STRIDE >= 0 && r - y * STRIDE < N)
                    acc[y] = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(A[r - y * STRIDE][t], B[t], acc[y], 0, 0, 0);
    }
}

// rows of nq quads one behind the other
template <int N, int STRIDE, int RO>
__device__ __forceinline__ void band_rows(f32x4_t (&acc)[RO], const short4_t (&A)[N][band_steps(N, STRIDE)], const char* p, int nq) {
    band_rows_at<N, STRIDE, RO>(acc, A, p, [nq](int r) { return r * nq * 8; });
}

// Batch-norm, activation and rounding of a strip's outputs: o[y] = four packed bf16 of row y.
// A band's zeros meet up to three pixels on either side of the taps, and a zero times an infinity or a NaN is NaN.  So the
// rounded outputs are multiplied with zeros once more (a matrix instruction a row, the vector units are what is short); the
// result is zero in every lane whose outputs are all finite.  The others -- strips of one channel -- have to be summed again
// (band_exact), after the stores, so that nothing waits for the check: 256 images of DS-MBNet 1016 -> 1018 us with the check
// there, 1003 after 992 with the check in front of the stores.
template <int RO>
__device__ __forceinline__ float band_finish(uint2 (&o)[RO], const f32x4_t (&acc)[RO], float sc, float sh, bool relu) {
    const short4_t none = {0, 0, 0, 0};
    f32x4_t chk = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int y = 0; y < RO; ++y) {
        o[y] = make_uint2(f2bf2(acc[y][0] * sc + sh, acc[y][1] * sc + sh), f2bf2(acc[y][2] * sc + sh, acc[y][3] * sc + sh));
        chk = __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(none, __builtin_bit_cast(short4_t, o[y]), chk, 0, 0, 0);
        if (relu) {
            // a positive bf16 is a positive 16-bit integer
            typedef __attribute__((ext_vector_type(2))) short short2_t;
            const short2_t zero = {0, 0};
            o[y].x = __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(short2_t, o[y].x), zero));
            o[y].y = __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(short2_t, o[y].y), zero));
        }
    }
    return chk[0];
}

// the same outputs tap by tap; weight(i, j): the channel's filter; p, at: as for band_rows_at
template <int N, int STRIDE, int RO, typename Weight, typename At>
__device__ __forceinline__ void band_exact_at(uint2 (&o)[RO], float sc, float sh, bool relu, Weight weight, const char* p, At at) {
#pragma unroll
    for (int y = 0; y < RO; ++y) {
        float v[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
        for (int t = 0; t < N * N; ++t) {
            const int i = t / N, j = t - i * N;
            const float w = bf2f(weight(i, j));
            const bf16_t* px = (const bf16_t*)(p + at(y * STRIDE + i)) + j;
#pragma unroll
            for (int k = 0; k < 4; ++k) v[k] = fmaf(w, bf2f(px[k * STRIDE]), v[k]);
        }
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            v[k] = v[k] * sc + sh;
            if (relu) v[k] = fmaxf(v[k], 0.f);
        }
        o[y] = make_uint2(f2bf2(v[0], v[1]), f2bf2(v[2], v[3]));
    }
}

// f: as for band_operand; rows of nq quads one behind the other
template <int N, int STRIDE, int RO>
__device__ __forceinline__ void band_exact(uint2 (&o)[RO], float sc, float sh, bool relu, const char* f, const char* p, int nq) {
    band_exact_at<N, STRIDE, RO>(o, sc, sh, relu, [f](int i, int j) { return ((const bf16_t*)f)[i * band_row_dwords(STRIDE) * 2 + band_lead(STRIDE) + j]; }, p,
                                 [nq](int r) { return r * nq * 8; });
}

// Four outputs of a channel after batch-norm and activation -> two of the channel pair: the lane trades half of them with
// its neighbour channel's lane of the same strip (lane 7 - i of 8: odd channels go over the strips backwards).  .x, .y: the
// pair (even channel low) at outputs 0, 1 of an even channel's lane, 2, 3 of an odd one's.
__device__ __forceinline__ uint2 band_trade(uint2 v, bool odd) {
    const uint32_t own = odd ? v.y : v.x, give = odd ? v.x : v.y;
    const uint32_t got = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)give, 0x141, 0xf, 0xf, true);
    const uint32_t x = odd ? 0x01000504u : 0x05040100u;    // bytes 0..3 of own, 4..7 of got
    return make_uint2(__builtin_amdgcn_perm(got, own, x), __builtin_amdgcn_perm(got, own, x + 0x02020202u));
}

// four pixels of 8 channels -> a quad of each channel
__device__ __forceinline__ void band_store_quads(char* t, int pitch, const uint4 (&px)[4]) {
    const uint32_t *p0 = &px[0].x, *p1 = &px[1].x, *p2 = &px[2].x, *p3 = &px[3].x;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        *(uint2*)(t + 2 * q * pitch) = make_uint2(__builtin_amdgcn_perm(p1[q], p0[q], 0x05040100), __builtin_amdgcn_perm(p3[q], p2[q], 0x05040100));
        *(uint2*)(t + (2 * q + 1) * pitch) = make_uint2(__builtin_amdgcn_perm(p1[q], p0[q], 0x07060302), __builtin_amdgcn_perm(p3[q], p2[q], 0x07060302));
    }
}
#endif
