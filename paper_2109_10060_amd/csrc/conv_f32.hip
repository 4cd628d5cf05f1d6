// fp32 NCHW sliced convolution on the fp32 matrix cores (single dynamic block, Section 3.3 Eq. 9 and Eq. 14).
//
// Bound: fp32 matrix rate for large batches (157 TFLOP/s nominal), latency for small ones.  A workgroup owns
// 32 filters x 32 consecutive output pixels of one sample and deals the input channels, CS at a time, to its four
// wavefronts: at 8 x 256 pixels x 64 channels there are about a hundred such tiles, so a tile's 576-step reduction has to
// be cut to be short.  A wavefront fetches the weights of its channel slice with 16-byte loads (a filter's taps are
// contiguous in memory) and turns them into matrix operands through an LDS region of its own -- no workgroup barrier
// before the final sum -- while the input goes straight into operand registers: pixels are the columns of
// v_mfma_f32_32x32x2_f32, so 32 lanes read 32 neighbouring pixels of a channel plane and the two lane halves take two
// channels.  All loads of a slice are requested before the first is used.  The four partial tiles are added in LDS in
// wavefront order; every lane then stores four results of one pixel column (128-byte runs over the lanes).
// The kernel finds a slot's route group in the offsets itself, so no slot table has to be built first.
// Padding is zeros that are multiplied, as in every other convolution here except conv_f32_kernel, which skips it: with a
// weight that is not finite the outputs at the border are NaN.
#include "common.h"

namespace {

// KS: filter size (1 or 3); CS: channels of a slice (even)
template <int KS, int CS>
__global__ __launch_bounds__(256, 2) void conv_f32_mfma_kernel(const float* x, const float* w, const float* scale,
                                                               const float* shift, int tab_ld, const float* residual,
                                                               float* y, const int32_t* offsets, const int32_t* perm,
                                                               const GroupTable gt, int C_I, int C_O, int H, int W, int Ho,
                                                               int Wo, int stride, int pad, int act, int n_ptiles,
                                                               int n_otiles, int wvec) {
    constexpr int KK = KS * KS, KN = CS * KK;              // reduction steps of a slice
    // row pitch in LDS: 2 modulo 4, so the 32 filter rows start on 32 distinct even banks and the other half of the
    // lanes, one channel (KK taps, odd) further, on the odd ones
    constexpr int LD = KN + ((KN & 3) == 0 ? 2 : 0);
    static_assert((LD & 3) == 2 && (KN & 3) == 0, "LDS pitch");
    constexpr int W_BYTES = 4 * 32 * LD * 4, R_BYTES = 4 * 16 * 64 * 4;
    __shared__ __attribute__((aligned(16))) char smem[W_BYTES > R_BYTES ? W_BYTES : R_BYTES];
    constexpr uint32_t OOB = 0x80000000u;

    const int bid = blockIdx.x;
    const int pt = bid % n_ptiles, ot = (bid / n_ptiles) % n_otiles, slot = bid / (n_ptiles * n_otiles);
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, l32 = lane & 31, lhi = lane >> 5;
    // group of the slot: the number of groups that end at or before it (T <= 64)
    const bool past = lane < gt.T && offsets[lane + 1] <= slot;
    const int g = __builtin_popcountll(__ballot(past));
    if (g >= gt.T) return;
    const int c_in = gt.k_in[g], k_out = gt.k_out[g];
    const int o0 = ot * 32;
    if (o0 >= k_out) return;
    const int b = perm ? perm[slot] : slot;
    const int px = pt * 32 + l32;
    const bool pok = px < Ho * Wo;
    const int oy = px / Wo, ox = px - oy * Wo;

    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc((void*)(x + (int64_t)b * C_I * H * W), 0, 0x7fffffff, 0x00020000);
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc((void*)w, 0, 0x7fffffff, 0x00020000);
    uint32_t off[KK];                                      // input pixel of each tap, channel lhi; OOB outside the image
#pragma unroll
    for (int t = 0; t < KK; ++t) {
        const int iy = oy * stride - pad + t / KS, ix = ox * stride - pad + t % KS;
        off[t] = pok && iy >= 0 && iy < H && ix >= 0 && ix < W ? (uint32_t)((lhi * H * W + iy * W + ix) * 4) : OOB;
    }
    float* wl = (float*)smem + wave * 32 * LD;
    f32x16_t acc;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0.f;

    const int wrow = C_I * KK;                             // floats of a stored filter
    for (int c0 = wave * CS; c0 < c_in; c0 += 4 * CS) {
        const int kn = min(CS, c_in - c0) * KK;            // valid reduction steps of the slice
        // ---- weights of 32 filters: four lanes read 64 consecutive bytes of a row, 16 rows at a time
        constexpr int PPR = KN / 4, NI = (PPR + 3) / 4;    // 16-byte pieces per row and per lane
        const int wq = lane & 3, wr = lane >> 2;
        float4 wv[2][NI];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int r = wr + 16 * j;
            const uint32_t wo = o0 + r < k_out ? (uint32_t)(((o0 + r) * wrow + c0 * KK + wq * 4) * 4) : OOB;
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const int k = wq * 4 + 16 * i;
                if (wvec) {
                    const auto q = __builtin_amdgcn_raw_buffer_load_b128(rw, (int)(k < kn ? wo : OOB), 64 * i, 0);
                    wv[j][i] = make_float4(__uint_as_float(q[0]), __uint_as_float(q[1]), __uint_as_float(q[2]), __uint_as_float(q[3]));
                } else {
                    float t[4];
#pragma unroll
                    for (int c = 0; c < 4; ++c)
                        t[c] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rw, (int)(k + c < kn ? wo : OOB), 64 * i + 4 * c, 0));
                    wv[j][i] = make_float4(t[0], t[1], t[2], t[3]);
                }
            }
        }
        // ---- input: one float per lane, tap and channel pair
        float xv[CS / 2][KK];
#pragma unroll
        for (int cp = 0; cp < CS / 2; ++cp) {
            const bool cok = c0 + 2 * cp + lhi < c_in;
#pragma unroll
            for (int t = 0; t < KK; ++t)
                xv[cp][t] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rx, (int)(cok ? off[t] : OOB), (c0 + 2 * cp) * H * W * 4, 0));
        }
        // a piece that reaches past the slice holds weights of channels beyond it: they enter as zeros
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int i = 0; i < NI; ++i) {
                const int k = wq * 4 + 16 * i;
                if (k >= KN) continue;
                float4 q = wv[j][i];
                if (k + 1 >= kn) q.y = 0.f;
                if (k + 2 >= kn) q.z = 0.f;
                if (k + 3 >= kn) q.w = 0.f;
                float* d = wl + (wr + 16 * j) * LD + k;
                *(float2*)d = make_float2(q.x, q.y);
                *(float2*)(d + 2) = make_float2(q.z, q.w);
            }
        // written and read by this wavefront alone: its LDS accesses complete in order
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        const float* wa = wl + l32 * LD + lhi * KK;
#pragma unroll
        for (int cp = 0; cp < CS / 2; ++cp)
#pragma unroll
            for (int t = 0; t < KK; ++t)
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(wa[2 * cp * KK + t], xv[cp][t], acc, 0, 0, 0);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    // ---- sum of the four partial tiles; wavefront q finishes accumulator rows 4 q .. 4 q + 3
    __syncthreads();
    float* red = (float*)smem;                             // [wavefront][16][64]
#pragma unroll
    for (int e = 0; e < 16; ++e) red[(wave * 16 + e) * 64 + lane] = acc[e];
    __syncthreads();
    if (!pok) return;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        const int e = wave * 4 + i;
        const int o = o0 + 8 * (e >> 2) + 4 * lhi + (e & 3);
        if (o >= k_out) continue;
        float v = red[e * 64 + lane];
#pragma unroll
        for (int q = 1; q < 4; ++q) v += red[(q * 16 + e) * 64 + lane];
        const int64_t ti = (int64_t)gt.row[g] * tab_ld + o;
        v = v * (scale ? scale[ti] : 1.f) + (shift ? shift[ti] : 0.f);
        const int64_t yi = ((int64_t)b * C_O + o) * Ho * Wo + px;
        if (residual) v += residual[yi];
        if (act == DS_ACT_RELU) v = fmaxf(v, 0.f);
        y[yi] = v;
    }
}

}  // namespace

int32_t ds_launch_conv_f32_mfma(const float* x, const float* w, const float* scale, const float* shift, int32_t tab_ld,
                                const float* residual, float* y, const int32_t* offsets, const int32_t* perm,
                                const GroupTable& gt, int32_t B, int32_t C_I, int32_t C_O, int32_t H, int32_t W, int32_t K,
                                int32_t stride, int32_t pad, int32_t act, hipStream_t s) {
    if (K != 1 && K != 3) return DS_EUNSUPPORTED;
    // 32-bit byte offsets against the sample and against the weights
    if ((int64_t)C_I * H * W * 4 >= 0x7fffffffLL || (int64_t)C_O * C_I * K * K * 4 >= 0x7fffffffLL) return DS_EUNSUPPORTED;
    const int Ho = (H + 2 * pad - K) / stride + 1, Wo = (W + 2 * pad - K) / stride + 1;
    int kmax = 0, omax = 0;
    for (int t = 0; t < gt.T; ++t) {
        kmax = gt.k_in[t] > kmax ? gt.k_in[t] : kmax;
        omax = gt.k_out[t] > omax ? gt.k_out[t] : omax;
    }
    if (B <= 0 || omax <= 0) return DS_OK;
    const int pts = (Ho * Wo + 31) / 32, ots = (omax + 31) / 32;
    if ((int64_t)pts * ots * B > 0x7fffffffLL) return DS_EUNSUPPORTED;
    const int wvec = ds_aligned16(w) && (C_I * K * K) % 4 == 0;
    ProfScope prof(DS_K_GEMM_TAPS, s);
#define DS_CONV_F32(KS, CS)                                                                                            \
    hipLaunchKernelGGL((conv_f32_mfma_kernel<KS, CS>), dim3((unsigned)(pts * ots * B)), dim3(256), 0, s, x, w, scale, shift, \
                       tab_ld, residual, y, offsets, perm, gt, C_I, C_O, H, W, Ho, Wo, stride, pad, act, pts, ots, wvec)
    // 16 channels a slice keep one slice per wavefront at 64 channels; up to 32 channels take 8, so that all four work
    if (K == 3) {
        if (kmax > 32) DS_CONV_F32(3, 16);
        else DS_CONV_F32(3, 8);
    } else {
        DS_CONV_F32(1, 16);
    }
#undef DS_CONV_F32
    DS_CHECK_LAUNCH("fp32 conv (matrix cores)");
    return DS_OK;
}
