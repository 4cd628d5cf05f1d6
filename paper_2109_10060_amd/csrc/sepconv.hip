// Depthwise-separable block behind the gate (every sample its route's slices) in one kernel: 3x3 depthwise convolution
// (padding 1, stride 1 or 2) + split batch-norm + ReLU feeding the 1x1 pointwise convolution + split batch-norm + ReLU
// (Section 3.2, Eq. 9, 10 and 14).  The depthwise map stays in the compute unit.
//
// As two launches a block moved that map through memory, the pointwise layer read it once per 64 filters, and with few samples
// two launches are two chains of latencies.  Here a workgroup owns some rows of one sample's map (16 RF pixels at most) and a run
// of 256 NP filters:
//   depthwise   a lane keeps one octet of channels, its nine taps and its batch-norm, and goes over strips of 4 (stride 2: 2)
//               neighbouring outputs: window straight from memory, products on channel pairs as in dwconv4_kernel (the same
//               bits), rounded into the operand tile [pixel][channel] in LDS;
//   pointwise   a wavefront owns NP times 32 filters; weights in operand order (16 filters x 32 channels = 1 KiB) straight into
//               registers, two steps in flight and the first ones under way during the depthwise part; the outputs replace the
//               operand tile and leave as whole lines.
// Channels past the slice are zeros in the tile, up to whole turns of 64, and the weights there are not read.
// Bound at full batches: the vector ALU in the depthwise part (9 of a full-width tile's 26 us), the matrix pipe behind it (8), and
// memory at both ends, one after the other with a workgroup a compute unit; with a few samples the chain of a workgroup.
// DS-MBNet, depthwise + pointwise launch before -> here, us: 14x14, 176..512 channels, one image 3.8 + 5.1 -> 5.0, 16 images
// 5.5 + 10.8 -> 9.6, 256 images 20.5 + 33.5 -> 40; 7x7, 360..1024 channels, 256 images 12.6 + 29.8 -> 41.7.
#include <algorithm>
#include <type_traits>

#include "common.h"

namespace {

constexpr uint32_t OOB = 0x80000000u;
constexpr int NW = 8;             // wavefronts of a workgroup

struct SepArgs {
    const bf16_t* x;
    const int32_t* xi;            // slot -> sample (nullable)
    int64_t x_ss, y_ss;
    bf16_t* y;                    // [slot][pixel][k_out]
    const bf16_t *wd, *wp;        // [9][C]; operand tiles
    const float *sd, *hd, *sp, *hp;
    const int32_t* slot_group;    // nullable: one group
    int32_t x_ld, C, F, kb, H, W, Ho, Wo, B, RO, tiles, runs;
    GroupTable gt;
};

__host__ __device__ constexpr int turns(int k) { return (k + 63) & ~63; }

// RF fragments of 16 pixels, NP groups of 32 filters for every wavefront
template <int STRIDE, int RF, int NP>
__global__ __launch_bounds__(64 * NW, 2) void sepconv_kernel(const SepArgs a) {
    constexpr int PX = STRIDE == 1 ? 4 : 2, NCOL = (PX - 1) * STRIDE + 3, D = 2, RUN = 32 * NW * NP;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    float* bn = (float*)smem;                            // [2][RUN]
    bf16_t* As = (bf16_t*)(smem + 8 * RUN);              // [16 RF][pitch]; then the outputs [16 RF][RUN + 8]

    // eight slots side by side (a sample stays on one die), widest routes first
    const GroupLanes lanes(a.gt);
    const int j = (int)(blockIdx.x >> 3), per = a.tiles * a.runs, s8 = j / per, rest = j - s8 * per;
    const int slot = ((a.B + 7) & ~7) - 8 - s8 * 8 + (int)(blockIdx.x & 7);
    if (slot >= a.B) return;
    const int tile = rest / a.runs, run = rest - tile * a.runs;
    const bf16_t *x = a.x, *wd = a.wd, *wp = a.wp;
    const float *sd = a.sd, *hd = a.hd, *sp = a.sp, *hp = a.hp;
    bf16_t* y = a.y;
    int64_t x_ss = a.x_ss, y_ss = a.y_ss;
    int x_ld = a.x_ld, C = a.C, F = a.F, kb = a.kb, H = a.H, W = a.W, Ho = a.Ho, Wo = a.Wo, RO = a.RO;
    const int g = a.slot_group ? a.slot_group[slot] : 0;
    const int sample = a.xi ? a.xi[slot] : slot;
    ds_hold(x, wd, wp, sd, hd, sp, hp, y, x_ss, y_ss, x_ld, C, F, kb, H, W, Ho, Wo, RO);
    const int K = lanes.k_in(g), N = lanes.k_out(g), trow = lanes.row(g);
    if (K <= 0 || N <= 0) return;
    const int groups = (N + 31) >> 5, g0 = run * (RUN / 32);
    const int oy0 = tile * RO, rows = min(RO, Ho - oy0);
    if (g0 >= groups || rows <= 0) return;
    if (x_ld <= 0) x_ld = K;

    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, l16 = lane & 15, kq = lane >> 4;
    const int Kp = turns(K), pitch = Kp + 8, nk = (K + 31) >> 5;
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc((void*)wp, 0, 0x7fffffff, 0x00020000);

    // weights: step k of group q; lanes past the slice (and steps past the last) get zeros without traffic
    bf16x8_t ring[D][NP][2];
    auto weights = [&](bf16x8_t (&r)[2], int q, int k) {
        const uint32_t off = k * 32 + kq * 8 < K ? (uint32_t)(lane * 16) : OOB;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const auto t = __builtin_amdgcn_raw_buffer_load_b128(rw, (int)off, (q * kb + k) * 2048 + h * 1024, 0);
            r[h] = __builtin_bit_cast(bf16x8_t, t);
        }
    };
    // this wavefront's groups of the run: w, w + NW, ...
    int ng = 0;
#pragma unroll
    for (int c = 0; c < NP; ++c) ng += g0 + w + NW * c < groups;
#pragma unroll
    for (int s = 0; s < D; ++s)
#pragma unroll
        for (int c = 0; c < NP; ++c)
            if (c < ng) weights(ring[s][c], g0 + w + NW * c, s);
    // the run's batch-norm (zeros past the slice)
    for (int i = tid; i < 2 * RUN; i += 64 * NW) {
        const int f = g0 * 32 + (i < RUN ? i : i - RUN);
        bn[i] = f < N ? (i < RUN ? sp : hp)[(int64_t)trow * F + f] : 0.f;
    }

    // ---- depthwise ----------------------------------------------------------------------------------------------------------
    {
        const int noct = Kp >> 3, side = 64 * NW / noct;         // strips at a time (Kp <= 512 NW: at least one)
        const int sl = tid / noct, oct = tid - sl * noct, ch = oct * 8;
        const int xg = (Wo + PX - 1) / PX, strips = rows * xg;
        const bool in = ch < K;
        if (sl < side) {
            const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc((void*)(x + (int64_t)sample * x_ss), 0, H * W * x_ld * 2, 0x00020000);
            constexpr uint32_t FAR = 0x40000000u;            // past any map, also twice
            uint4 win[9];
            float sc[8], sh[8];
            if (in) {
                const int64_t ti = (int64_t)trow * C + ch;
#pragma unroll
                for (int t = 0; t < 9; ++t) win[t] = *(const uint4*)(wd + t * C + ch);
#pragma unroll
                for (int i = 0; i < 8; i += 4) {
                    *(float4*)(sc + i) = *(const float4*)(sd + ti + i);
                    *(float4*)(sh + i) = *(const float4*)(hd + ti + i);
                }
            }
            for (int s = sl; s < strips; s += side) {
                const int r = s / xg, ox0 = (s - r * xg) * PX, oy = oy0 + r;
                bf16_t* out = As + (r * Wo + ox0) * pitch + ch;
                if (!in) {
#pragma unroll
                    for (int p = 0; p < PX; ++p)
                        if (ox0 + p < Wo) *(uint4*)(out + p * pitch) = make_uint4(0, 0, 0, 0);
                    continue;
                }
                uint4 xin[3][NCOL];
                uint32_t ro[3];
#pragma unroll
                for (int u = 0; u < 3; ++u) {
                    const int iy = oy * STRIDE + u - 1;
                    ro[u] = (unsigned)iy < (unsigned)H ? (uint32_t)(iy * W * x_ld + ch) * 2 : FAR;
                }
#pragma unroll
                for (int col = 0; col < NCOL; ++col) {
                    const int ix = ox0 * STRIDE - 1 + col;
                    const uint32_t co = (unsigned)ix < (unsigned)W ? (uint32_t)(ix * x_ld) * 2 : FAR;
#pragma unroll
                    for (int u = 0; u < 3; ++u) {
                        const auto t = __builtin_amdgcn_raw_buffer_load_b128(rx, (int)(ro[u] + co), 0, 0);
                        xin[u][col] = make_uint4(t[0], t[1], t[2], t[3]);
                    }
                }
                float acc[PX][8];
#pragma unroll
                for (int p = 0; p < PX; ++p)
#pragma unroll
                    for (int i = 0; i < 8; ++i) acc[p][i] = 0.f;
#pragma unroll
                for (int u = 0; u < 3; ++u) {
                    bf16x2_t wlo[3][4], whi[3][4];
#pragma unroll
                    for (int v = 0; v < 3; ++v) {
                        const uint32_t qq[4] = {win[u * 3 + v].x, win[u * 3 + v].y, win[u * 3 + v].z, win[u * 3 + v].w};
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            wlo[v][i] = __builtin_bit_cast(bf16x2_t, qq[i] & 0x0000ffffu);
                            whi[v][i] = __builtin_bit_cast(bf16x2_t, qq[i] & 0xffff0000u);
                        }
                    }
#pragma unroll
                    for (int col = 0; col < NCOL; ++col) {
                        const uint4 q = xin[u][col];
                        const bf16x2_t xq[4] = {__builtin_bit_cast(bf16x2_t, q.x), __builtin_bit_cast(bf16x2_t, q.y),
                                                __builtin_bit_cast(bf16x2_t, q.z), __builtin_bit_cast(bf16x2_t, q.w)};
#pragma unroll
                        for (int p = 0; p < PX; ++p) {
                            const int v = col - p * STRIDE;
                            if (v >= 0 && v < 3) {
#pragma unroll
                                for (int i = 0; i < 4; ++i) {
                                    acc[p][2 * i] = __builtin_amdgcn_fdot2_f32_bf16(xq[i], wlo[v][i], acc[p][2 * i], false);
                                    acc[p][2 * i + 1] = __builtin_amdgcn_fdot2_f32_bf16(xq[i], whi[v][i], acc[p][2 * i + 1], false);
                                }
                            }
                        }
                    }
                }
#pragma unroll
                for (int p = 0; p < PX; ++p) {
                    if (ox0 + p >= Wo) break;
                    float v[8];
#pragma unroll
                    for (int i = 0; i < 8; ++i) v[i] = fmaxf(acc[p][i] * sc[i] + sh[i], 0.f);
                    *(uint4*)(out + p * pitch) = make_uint4(f2bf2(v[0], v[1]), f2bf2(v[2], v[3]), f2bf2(v[4], v[5]), f2bf2(v[6], v[7]));
                }
            }
        }
    }
    __syncthreads();

    // ---- pointwise ----------------------------------------------------------------------------------------------------------
    const int px = rows * Wo, spitch = NW * NP * 32 + 8;
    auto products = [&](auto n) {
        constexpr int NN = decltype(n)::value;
        f32x4_t acc[NN][2][RF];
#pragma unroll
        for (int c = 0; c < NN; ++c)
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int m = 0; m < RF; ++m) acc[c][h][m] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        for (int k0 = 0; k0 < nk; k0 += D) {
#pragma unroll
            for (int s = 0; s < D; ++s) {
                bf16x8_t pf[RF];
#pragma unroll
                for (int m = 0; m < RF; ++m) pf[m] = *(const bf16x8_t*)(As + (m * 16 + l16) * pitch + (k0 + s) * 32 + kq * 8);
#pragma unroll
                for (int c = 0; c < NN; ++c) {
#pragma unroll
                    for (int h = 0; h < 2; ++h)
#pragma unroll
                        for (int m = 0; m < RF; ++m)
                            acc[c][h][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ring[s][c][h], pf[m], acc[c][h][m], 0, 0, 0);
                    weights(ring[s][c], g0 + w + NW * c, k0 + s + D);
                }
            }
        }
        __syncthreads();                                 // the operand tile has been read: it becomes the output tile
#pragma unroll
        for (int c = 0; c < NN; ++c) {
            const int f = (w + NW * c) * 32 + kq * 8;
            float sc[8], sh[8];
#pragma unroll
            for (int i = 0; i < 8; i += 4) {
                *(float4*)(sc + i) = *(const float4*)(bn + f + i);
                *(float4*)(sh + i) = *(const float4*)(bn + RUN + f + i);
            }
#pragma unroll
            for (int m = 0; m < RF; ++m) {
                float v[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) v[i] = fmaxf(acc[c][i >> 2][m][i & 3] * sc[i] + sh[i], 0.f);
                *(uint4*)(As + (m * 16 + l16) * spitch + f) = make_uint4(f2bf2(v[0], v[1]), f2bf2(v[2], v[3]), f2bf2(v[4], v[5]), f2bf2(v[6], v[7]));
            }
        }
    };
    static_assert(NP <= 2, "");
    if (ng == NP) products(std::integral_constant<int, NP>{});
    else if (NP > 1 && ng == 1) products(std::integral_constant<int, 1>{});
    else __syncthreads();                                // no filters: the barrier inside
    __syncthreads();
    // rows of the tile are neighbours in memory: whole lines
    const int n0 = g0 * 32, cols8 = min(N - n0, RUN) >> 3, inv = (1 << 20) / cols8 + 1;
    bf16_t* yb = y + (int64_t)slot * y_ss + (int64_t)oy0 * Wo * N + n0;
    for (int e = tid; e < px * cols8; e += 64 * NW) {
        const int p = (int)(((int64_t)e * inv) >> 20), c = e - p * cols8;     // (e < 2^14, cols8 <= 64: exact)
        *(uint4*)(yb + (int64_t)p * N + c * 8) = *(const uint4*)(As + p * spitch + c * 8);
    }
}

template <int STRIDE, int RF, int NP>
int32_t launch(SepArgs& a, int kmax, int groups, hipStream_t s) {
    constexpr int RUN = 32 * NW * NP;
    const int most = RF * 16 / a.Wo;                     // rows of a tile
    const int smem = 8 * RUN + RF * 16 * (std::max(turns(kmax), RUN) + 8) * 2;
    if (most < 1 || smem > 160 * 1024) return DS_EUNSUPPORTED;
    a.tiles = (a.Ho + most - 1) / most;
    a.RO = (a.Ho + a.tiles - 1) / a.tiles;
    a.runs = (groups * 32 + RUN - 1) / RUN;
    const int64_t grid = (int64_t)((a.B + 7) / 8) * 8 * a.tiles * a.runs;
    if (grid > 0x7fffffff) return DS_EUNSUPPORTED;
    auto kern = sepconv_kernel<STRIDE, RF, NP>;
    const int32_t rc = ds_reserve_lds((const void*)kern, 160 * 1024, "sliced separable block");
    if (rc) return rc;
    ProfScope prof(DS_K_DWCONV, s);
    hipLaunchKernelGGL(kern, dim3((unsigned)grid), dim3(64 * NW), smem, s, a);
    DS_CHECK_LAUNCH("sliced separable block");
    return DS_OK;
}

// Pixels and filters of a workgroup.  Fewer of both mean more workgroups, each a shorter chain, but the weights come in once per tile
// and the depthwise part is done once per run of filters.  Measured on DS-MBNet, us a launch, 32 pixels and 256 filters / 32 and
// 512 / 64 and 512 / 112 and 512:
//   14x14, 512 -> 512    16 images 9.8 / 11.9 / 14.7 / -, 24 images 13.3 / 11.9 / 15.0 / -, 48 images 20.3 / 15.6 / 16.0 / -,
//                        64 images 26.9 / 18.2 / 16.6 / 22.8, 128 images 47.6 / 35.6 / 26.5 / 26.0, 256 images 89 / 61 / 48 / 40
//   7x7, 1024 -> 1024    24 images 13.2 / 17.5 / 23.0, 48 images 18.3 / 17.8 / 23.4, 64 images 21.4 / 18.4 / 23.5, 128 images 40.5 / 31.2 / 27.3
// so the smaller tile ends where its workgroups are one for every compute unit (a third more where only the tile grows), and 64
// pixels end at two.  Counted on the die that has the most, as a sample stays on one: of 17 samples it has three.  Against the same
// lines on the whole chip: 17 / 18 images 196.9 / 199.4 -> 191.8 / 192.9 us a pass, 9 to 256 others the same.
template <int STRIDE>
int32_t dispatch(SepArgs& a, int kmax, int groups, hipStream_t s) {
    // on the die with the most samples (32 compute units)
    auto tiles = [&](int rf) { return (int64_t)((a.B + 7) / 8) * ((a.Ho + rf * 16 / a.Wo - 1) / (rf * 16 / a.Wo)); };
    const int64_t t2 = tiles(2);
    const int r16 = (groups + 15) / 16;
    if (t2 * ((groups + 7) / 8) > 32) {
        int32_t rc = DS_EUNSUPPORTED;
        if (t2 * r16 > 42) {
            if (tiles(4) > 64 && a.Ho * a.Wo > 64) rc = launch<STRIDE, 7, 2>(a, kmax, groups, s);
            if (rc == DS_EUNSUPPORTED) rc = launch<STRIDE, 4, 2>(a, kmax, groups, s);
        }
        if (rc == DS_EUNSUPPORTED) rc = launch<STRIDE, 2, 2>(a, kmax, groups, s);
        if (rc != DS_EUNSUPPORTED) return rc;
    }
    return launch<STRIDE, 2, 1>(a, kmax, groups, s);
}

}  // namespace

int32_t ds_launch_sepconv(ActView x, bf16_t* y, int64_t y_ss, const bf16_t* wd, const float* sd, const float* hd, int32_t C, const bf16_t* wp,
                          const float* sp, const float* hp, int32_t F, const int32_t* slot_group, const GroupTable& gt, int32_t B,
                          int32_t H, int32_t W, int32_t stride, hipStream_t s) {
    if (B <= 0) return DS_OK;
    int kmax = 0, nmax = 0;
    for (int t = 0; t < gt.T; ++t) {
        kmax = std::max(kmax, (int)gt.k_in[t]);
        nmax = std::max(nmax, (int)gt.k_out[t]);
        if ((gt.k_in[t] % 8) || (gt.k_out[t] % 8)) return DS_EUNSUPPORTED;
    }
    if ((stride != 1 && stride != 2) || turns(C) > 2048 || (W - 1) / stride + 1 > 32) return DS_EUNSUPPORTED;
    if (kmax <= 0 || nmax <= 0) return DS_OK;
    SepArgs a = {};
    a.x = (const bf16_t*)x.p; a.xi = x.index; a.x_ss = x.sample_stride; a.x_ld = x.ld; a.y = y; a.y_ss = y_ss;
    a.wd = wd; a.wp = wp; a.sd = sd; a.hd = hd; a.sp = sp; a.hp = hp; a.slot_group = slot_group;
    a.C = C; a.F = F; a.kb = (C + 31) / 32 | 1; a.H = H; a.W = W; a.Ho = (H - 1) / stride + 1; a.Wo = (W - 1) / stride + 1; a.B = B;
    a.gt = gt;
    if ((int64_t)H * W * (x.ld > 0 ? x.ld : kmax) * 2 >= 0x40000000LL || (int64_t)((F + 31) / 32) * a.kb * 2048 >= 0x7fffffffLL) return DS_EUNSUPPORTED;
    const int groups = (nmax + 31) / 32;
    return stride == 1 ? dispatch<1>(a, kmax, groups, s) : dispatch<2>(a, kmax, groups, s);
}
