// Row helpers shared by the transformer-block kernels that keep a tile of token rows in LDS.
#pragma once

#include "common.h"

__device__ __forceinline__ void unpack8(const uint4 q, float* v) {
    const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        v[2 * i] = __uint_as_float(w[i] << 16);
        v[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
    }
}
__device__ __forceinline__ uint4 pack8(const float* v) {
    return make_uint4(f2bf2(v[0], v[1]), f2bf2(v[2], v[3]), f2bf2(v[4], v[5]), f2bf2(v[6], v[7]));
}

// sum over 16 neighbouring lanes, all of them get it: rotations within the row of 16, the same pairs as exchanges over lane bits 3, 2,
// 1, 0 (after the first step the values repeat every 8 lanes, then every 4, 2) and so the same bits, without LDS round trips
__device__ __forceinline__ float row16_sum(float s) {
    s += __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(s), 0x128, 0xf, 0xf, true));
    s += __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(s), 0x124, 0xf, 0xf, true));
    s += __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(s), 0x122, 0xf, 0xf, true));
    s += __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(s), 0x121, 0xf, 0xf, true));
    return s;
}
// LayerNorm of one row held by 16 lanes, lane l with the 8-channel chunks l, l + 16, l + 32, l + 48; the arithmetic and
// the order of layernorm16_kernel.  SKIP: chunks that begin behind the slice are skipped by a branch of the whole wavefront (a normalised row
// is about 450 vector instructions of a lane, and of the four chunks a slice of 192 or 256 channels has two).  Not with eight wavefronts in
// vit_linear_kernel: there the branches cost more than they save.  With them / without: the first block's Q/K/V layer of 256 images of DS-ViT++
// 63.8 / 62.6 us, passes of 1 / 3 images of DS-ViT 399.0 / 432.5 and 397.5 / 430.5 us.
template <bool SKIP>
__device__ __forceinline__ bool row_has(int k, int d) { return !SKIP || 128 * k < d; }
template <bool SKIP>
__device__ __forceinline__ float row_stats(const float (&v)[4][8], int d, int l16, float eps, float* mean) {
    float s = 0.f;
#pragma unroll
    for (int k = 0; k < 4; ++k)
        if (row_has<SKIP>(k, d)) if ((k * 16 + l16) * 8 < d) {
#pragma unroll
            for (int i = 0; i < 8; ++i) s += v[k][i];
        }
    const float mu = row16_sum(s) / (float)d;
    *mean = mu;
    float q = 0.f;
#pragma unroll
    for (int k = 0; k < 4; ++k)
        if (row_has<SKIP>(k, d)) if ((k * 16 + l16) * 8 < d) {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const float t = v[k][i] - mu;
                q += t * t;
            }
        }
    return 1.0f / sqrtf(row16_sum(q) / (float)d + eps);
}
template <bool SKIP = true>
__device__ __forceinline__ void row_norm(const float (&v)[4][8], int d, int l16, float eps, const float* gamma,
                                         const float* beta, uint4 (&out)[4]) {
    float mu;
    const float rstd = row_stats<SKIP>(v, d, l16, eps, &mu);
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int ch = (k * 16 + l16) * 8;
        if (row_has<SKIP>(k, d)) if (ch < d) {
            const float4 g0 = *(const float4*)(gamma + ch), g1 = *(const float4*)(gamma + ch + 4);
            const float4 b0 = *(const float4*)(beta + ch), b1 = *(const float4*)(beta + ch + 4);
            const float gm[8] = {g0.x, g0.y, g0.z, g0.w, g1.x, g1.y, g1.z, g1.w};
            const float bt[8] = {b0.x, b0.y, b0.z, b0.w, b1.x, b1.y, b1.z, b1.w};
            float o8[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) o8[i] = (v[k][i] - mu) * rstd * gm[i] + bt[i];
            out[k] = pack8(o8);
        }
    }
}

// Row pitch in elements of an activation tile of up to k channels that is multiplied in turns of d 16-channel steps: the row
// holds every step of the last turn, those past the slice as zeros (what follows in LDS is another sample's row, which need
// not be finite, and zero weights alone do not undo that).  An odd number of 16-byte chunks, so 32 rows read without conflicts.
__host__ __device__ constexpr int tile_pitch(int k, int d) { return (k + 16 * d - 1) / (16 * d) * (16 * d) + 8; }
constexpr int VIT_K_MAX = 416;      // channels of a row that is normalised or multiplied in one tile

// Weights in operand order: 1 KiB tiles of 32 rows x 16 channels, the upper 8 channels behind the lower ones.  A descriptor of
// the tiles of one row block from tile t0 on that ends with the slice of k channels (a multiple of 8): lanes past it get zeros
// without traffic, also the upper half of a slice's last step -- the stored weights go on there and need not be finite.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t weight_row(const bf16_t* w, int t0, int k) {
    return __builtin_amdgcn_make_buffer_rsrc((void*)(w + (int64_t)t0 * 512), 0, k * 64, 0x00020000);
}
// a whole kilobyte per wavefront; off: lane * 16 plus 1024 a tile
__device__ __forceinline__ bf16x8_t weight_tile(const __amdgpu_buffer_rsrc_t& rs, uint32_t off) {
    const auto q = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)off, 0, 0);
    return __builtin_bit_cast(bf16x8_t, q);
}
