// 3x3 layers (padding 1, bf16, no residual: conv3_kernel's of stride 1, and those of stride 2) with the filters in operand order: they stream into registers, and only the
// input patch, staged once a chunk of 32 channels, goes through LDS.  Sums in conv3_kernel's order: chunk, tap, half of the chunk
// (gemm_kernel takes a strided layer tap by tap, so the last bits differ where a batch's size sends one there).
//
// What bounds it: matrix rate, while a SIMD has two wavefronts.  One wavefront alone gets an instruction out of 61 clocks where the pipe takes 32: all four
// of a workgroup ask LDS and the vector cache at once, and its products wait behind the requests in program order (245 clocks a step of four products, with
// requests between the products; 258 with all of a step's reads ahead of them, whether or not anything comes from memory).  Two workgroups a compute unit
// take 156.  Measured on 256 images of 14x14 pixels on one route: 64 / 128 / 192 / 256 channels 314 / 655 / 776 / 996 TFLOP/s.
//   * A wavefront has 32 filters and all 128 pixels of a tile (64 of 64): a filter operand serves four products, so that LDS (four wavefronts read the same
//     pixels) and the vector cache (each its own filters) both stay below what they deliver; two blocks of filters by 64 pixels 41 us where this takes 39.
//   * Padded pixels (conv3_fit.h): with masks and a row of zeros each operand cost four vector instructions, with zeros in place none.
//   * DS steps of filters are on their way.  An input patch is asked for a chunk ahead; its loads return in order with the filters'.
//   * A launch is one or two generations, and workgroups b and b + 256 start on the same compute unit: the first 32 of a die are dealt from the 32nd widest
//     to the widest, so that the widest ones share with the narrowest or with none.  A row tile stays on the die that gemm_kernel's layers in front and
//     behind have it on: with tiles dealt over all dies the 3x3 layers of DS-ResNet took 13 us less each and the pass nothing less.
//   * Quotients by reciprocals: with integer divisions a workgroup spent 14 of 25 us ahead of its first product and behind its last.
// us a launch, mixed routes of 256 images, conv3_kernel -> here: 14x14 pixels, 64..256 channels 46 -> 32, 7x7 pixels, 128..512 channels 46 -> 32.
// us a pass, without this kernel | its layers of stride 1 | all of them (one card, in turn, a second each): DS-ResNet 8 / 16 / 24 / 33 / 48 images 521 / 611 / 681 / 747 / 872 |
// 516 / 597 / 654 / 699 / 841 | 516 / 594 / 646 / 690 / 822, 64 / 96 / 128 / 160 / 256 images 1026 / 1224 / 1477 / 1693 / 2434 | 1000 / 1183 / 1425 / 1635 / 2339 | 976 / 1156 / 1395 /
// 1609 / 2327, 256 in four parts 2422 | 2344 | 2318, DS-ResNet++ 8 / 16 / 33 / 64 / 128 / 256 images 514 / 601 / 775 / 1099 / 1646 / 2776 | 507 / 583 / 729 / 1067 / 1581 / 2677 | 505 / 579 / 714 /
// 1039 / 1547 / 2637.  Of the 125 us that the launches of 256 images save under events the pass keeps 107; on cards of lower clocks it kept 30 to 65 (2478 -> 2449, 2494 -> 2429).
// Three networks in turn, so that filters come from memory: DS-ResNet 16 / 24 / 33 / 48 / 256 images 650 / 723 / 798 / 917 / 2434 | 653 / 711 / 776 / 900 / 2338 | 653 / 706 / 773 / 890 / 2326,
// DS-ResNet++ 33 images 825 | 811 | 802.
#include "tile_out.h"
#include "conv3_fit.h"

namespace {

constexpr int BN = 128;
constexpr int PITCH = CONV3_PITCH;
constexpr int CHUNK = 18;                      // steps of a chunk: 9 taps of two 16-channel halves
constexpr int FOLD = 32;                       // compute units of a die
constexpr int patch_bytes(int stride, int bm) { return stride == 2 ? CONV3_BYTES2 : conv3_bytes(bm); }
constexpr int smem_bytes(int stride, int bm) { return 2 * patch_bytes(stride, bm) + 2 * BN * 4; }
constexpr uint32_t OOB = 0x80000000u;

struct Conv3T {
    const bf16_t* w;                           // [ceil(N / 32)][ntile] tiles of 1 KiB
    int32_t ntile;                             // 18 a chunk and one that keeps the blocks' streams off the same L2 channels
};

// CW of the four wavefronts side by side, 32 filters each, 4 / CW below each other, 32 R pixels each; DS steps of filters on their way, pixels read FA - 1 steps ahead
template <int S, int R, int CW, int DS, int FA>
__device__ __forceinline__ void body(const GemmArgs& a, const Conv3T& t, const int g0, const int slot0, const int rows_g, const int n0, const int k_in, const int k_out, const int row, char* smem) {
    constexpr int NW = 4, RW = NW / CW, BM = 32 * R * RW, RMAX = S == 2 ? CONV3_PIXELS2 : conv3_pixels(BM), PB = patch_bytes(S, BM), NT = 64 * NW, NI = (RMAX + 16 * NW - 1) / (16 * NW), NC = (NI + 3) / 4;
    static_assert(CHUNK % DS == 0 && CHUNK % FA == 0, "whole turns");
    float* scl = (float*)(smem + 2 * PB);    // [BN] scale, then [BN] shift
    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, l32 = lane & 31, lhi = lane >> 5;
    const int cw = w % CW, rw = w / CW;
    const int W = a.W, H = a.H, Wo = a.Wo, Q = S == 2 ? conv3_pitch2(W) : W + 1, rows = a.rows;
    const float r_rows = __builtin_amdgcn_rcpf((float)rows), r_w = __builtin_amdgcn_rcpf((float)Wo), r_q = __builtin_amdgcn_rcpf((float)Q), r_h = __builtin_amdgcn_rcpf((float)(H + 1));
    static_assert(NT >= BN, "a lane a column");
    float vs = 1.f, vh = 0.f;
    if (tid < BN && n0 + tid < k_out) {
        const long long ti = (long long)row * a.tab_ld + n0 + tid;
        if (a.scale) vs = a.scale[ti];
        if (a.shift) vh = a.shift[ti];
    }
    const int a_ld = a.a_ld > 0 ? a.a_ld : k_in, c_ld = a.c_ld > 0 ? a.c_ld : k_out;
    const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc((void*)a.A, 0, 0x7fffffff, 0x00020000);
    const int blk = n0 / 32 + cw;
    const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc((void*)(t.w + (int64_t)blk * t.ntile * 512), 0, blk * 32 < k_out ? t.ntile * 1024 : 0, 0x00020000);
    const uint32_t lane16 = (uint32_t)lane * 16;
    const int nchunk = (k_in + 31) / 32;
    // padded index of tap (0, 0) of a pixel
    auto padded = [&](int m) {
        const int sl = quotient22(m, rows, r_rows), p = m - sl * rows, y = quotient22(p, Wo, r_w);
        return S == 2 ? conv3_padded2(sl, y, p - y * Wo, W, H) : conv3_padded(sl, y, p - y * W, W, H) - (Q + 1);
    };
    const int first = padded(g0), span = padded(min(g0 + BM, rows_g) - 1) + 2 * Q + 3 - first;
    const int RB = W * PITCH + CONV3_GAP, row0 = S == 2 ? 0 : quotient22(first, Q, r_q);
    uint32_t poff[NI];
    int loff[NI];
    {
        uint32_t o[NC], l[NC];
#pragma unroll
        for (int k = 0; k < NC; ++k) {
            const int j = 16 * w + 16 * NW * (4 * k + (lane >> 4)) + (lane & 15), P = first + j;
            const int pr = quotient22(P, Q, r_q), x = P - pr * Q - 1, sl = quotient22(pr, H + 1, r_h), y = pr - sl * (H + 1) - 1, p = y * W + x;
            o[k] = OOB;
            l[k] = (uint32_t)(j < span ? (S == 2 ? conv3_byte2(P, first) : conv3_byte(pr, x + 1, row0, W)) : -1);
            if (j < span && x >= 0 && x < W && y >= 0 && sl * rows < rows_g) {
                const int slot = slot0 + sl, sa = a.a_index ? a.a_index[slot] : slot;
                o[k] = ((uint32_t)sa * (uint32_t)a.a_sample_stride + (uint32_t)(p * a_ld)) * 2;
            }
        }
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const uint32_t q = (uint32_t)__shfl((int)o[i / 4], (i & 3) * 16 + (lane >> 2), 64);
            poff[i] = q == OOB ? OOB : q + (lane & 3) * 16;
            const int d = __shfl((int)l[i / 4], (i & 3) * 16 + (lane >> 2), 64);
            loff[i] = d < 0 ? -1 : d + (lane & 3) * 16;
        }
    }
    uint4 pv[NI];
    auto load_patch = [&](int c) __attribute__((always_inline)) {
        const bool ok = c * 32 + (lane & 3) * 8 < k_in;
#pragma unroll
        for (int i = 0; i < NI; ++i) pv[i] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(ra, (int)(ok ? poff[i] : OOB), c * 64, 0));
    };
    auto store_patch = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NI; ++i)
            if (loff[i] >= 0) *(uint4*)(smem + buf * PB + loff[i]) = pv[i];
    };
    if constexpr (S == 1) {
        // the zeros behind a map row (those ahead of it come with the patch)
        const int nrow = quotient22(first + span - 1, Q, r_q) - row0 + 1;
        for (int i = tid; i < nrow * 8; i += NT)
            *(uint4*)(smem + (i >> 2 & 1) * PB + (i >> 3) * RB + (W + 1) * PITCH + (i & 3) * 16) = make_uint4(0, 0, 0, 0);
    }
    bf16x8_t ring[DS];
    uint32_t vo[2], vn[2];                             // of the chunk at hand, of the next one: nothing behind the slice
    auto reach = [&](uint32_t (&v)[2], int c) {
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) v[kk] = c * 32 + kk * 16 + lhi * 8 < k_in ? lane16 : OOB;
    };
    auto ask = [&](int s, const uint32_t (&v)[2], int c) __attribute__((always_inline)) {      // step s of chunk c
        ring[s % DS] = __builtin_bit_cast(bf16x8_t, __builtin_amdgcn_raw_buffer_load_b128(rb, (int)v[s & 1], (c * CHUNK + s) * 1024, 0));
    };
    load_patch(0);
    reach(vo, 0);
#pragma unroll
    for (int s = 0; s < DS; ++s) ask(s, vo, 0);
    if (tid < BN) {
        scl[tid] = vs;
        scl[BN + tid] = vh;
    }
    int base[R];                                       // byte of tap (0, 0) of this lane's pixels
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int m = g0 + (rw * R + r) * 32 + l32;
        const int P = m < rows_g ? padded(m) : first, pr = S == 2 ? 0 : quotient22(P, Q, r_q);
        base[r] = (S == 2 ? conv3_byte2(P, first) : conv3_byte(pr, P - pr * Q, row0, W)) + lhi * 16;
    }
    f32x16_t acc[R];
#pragma unroll
    for (int r = 0; r < R; ++r)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[r][v] = 0.f;
    store_patch(0);
    __syncthreads();
    for (int c = 0; c < nchunk; ++c) {
        const char* cur = smem + (c & 1) * PB;
        reach(vn, c + 1);
        bf16x8_t f[FA][R];
        auto read = [&](int s, int r) __attribute__((always_inline)) {
            const int u = s / 6, v = s / 2 % 3, kk = s & 1;
            f[s % FA][r] = *(const bf16x8_t*)(cur + base[r] + (S == 2 ? conv3_tap2(u, v, W) : u * RB + v * PITCH) + kk * 32);
        };
#pragma unroll
        for (int s = 0; s < FA - 1; ++s)
#pragma unroll
            for (int r = 0; r < R; ++r) read(s, r);
        load_patch(c + 1);                             // (behind the slice: nothing)
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int s = 0; s < CHUNK; ++s) {
#pragma unroll
            for (int r = 0; r < R; ++r) {
                acc[r] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[s % DS], f[s % FA][r], acc[r], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                if (s + FA - 1 < CHUNK) read(s + FA - 1, r);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (s + DS < CHUNK) ask(s + DS, vo, c);
            else ask(s + DS - CHUNK, vn, c + 1);
            __builtin_amdgcn_sched_barrier(0);
        }
        store_patch((c + 1) & 1);
        vo[0] = vn[0], vo[1] = vn[1];
        __syncthreads();
    }
    // ---- a lane holds channels 8 q + 4 lhi .. + 3 of its pixels: traded between the wavefront's halves, 16 bytes a store
    with_act<false>(a.act, [&](auto actc) {
        constexpr int ACT = decltype(actc)::value;
        bf16_t* out[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int m = g0 + (rw * R + r) * 32 + l32, sl = m < rows_g ? quotient22(m, rows, r_rows) : 0, p = m - sl * rows, slot = slot0 + sl;
            const int cs = a.c_index ? a.c_index[slot] : slot;
            out[r] = m < rows_g ? (bf16_t*)a.C + (long long)cs * a.c_sample_stride + (long long)(p + a.c_row0) * c_ld : nullptr;
        }
#pragma unroll
        for (int q = 0; q < 4; q += 2) {
            const float* sp = scl + cw * 32 + 8 * q + 4 * lhi;
            const float4 s4[2] = {*(const float4*)sp, *(const float4*)(sp + 8)}, h4[2] = {*(const float4*)(sp + BN), *(const float4*)(sp + BN + 8)};
            const int n = n0 + cw * 32 + 8 * q + 8 * lhi;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                uint2 o[2];
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const int i = 4 * (q + e);
                    const f32x16_t& v = acc[r];
                    float val[4] = {v[i] * s4[e].x + h4[e].x, v[i + 1] * s4[e].y + h4[e].y, v[i + 2] * s4[e].z + h4[e].z, v[i + 3] * s4[e].w + h4[e].w};
                    o[e] = activate_bf16<ACT>(val);
                }
                const auto lo = __builtin_amdgcn_permlane32_swap(o[0].x, o[1].x, false, false);
                const auto hi = __builtin_amdgcn_permlane32_swap(o[0].y, o[1].y, false, false);
                if (out[r] && n < k_out) *(uint4*)(out[r] + n) = make_uint4(lo[0], hi[0], lo[1], hi[1]);
            }
        }
    });
}

template <int S, int BM>
__global__ __launch_bounds__(256, 2) void conv3_tiled_kernel(const GemmArgs a, const Conv3T t) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const GroupLanes lanes(a.gt);
    const int32_t* offsets = a.offsets;
    int T = a.gt.T, rows = a.rows;
    ds_hold(offsets, T, rows);
    // ---- this die's tiles, widest slices first: row tile m of 128 rows, counted over the groups as gemm_kernel does, is die m % 8's, as in the
    // layers in front and behind, which leave and look for its rows in that die's L2.  Lane i counts those of group T - 1 - i.
    const int lane = threadIdx.x & 63, gi = T - 1 - lane, at = gi >= 0 ? gi : 0, die = (int)blockIdx.x & 7, b = (int)blockIdx.x >> 3;
    const int o0 = offsets[at], o1 = offsets[at + 1];
    const int ki = __shfl(lanes.ki, at, 64), ko = __shfl(lanes.ko, at, 64);
    const int nm = gi >= 0 ? ((o1 - o0) * rows + DS_GEMM_BM - 1) / DS_GEMM_BM : 0, mend = ds_scan64(nm);
    const int k0 = (mend - nm + 7 - die) >> 3, mine = ((mend + 7 - die) >> 3) - k0;      // of this die: ahead of the group, in it
    const int parts = (DS_GEMM_BM / BM) * ((ko + BN - 1) / BN);                          // workgroups of a row tile
    const int cnt = ki > 0 && ko > 0 ? mine * parts : 0, upto = ds_scan64(cnt), total = __builtin_amdgcn_readlane(upto, 63);
    if (b >= total) return;
    const int rank = b < FOLD ? min(FOLD, total) - 1 - b : b;
    const int q = __builtin_ctzll(__ballot(upto > rank));
    const int i = rank - __builtin_amdgcn_readlane(upto - cnt, q), np = __builtin_amdgcn_readlane(parts, q);
    const int k = ds_quotient_uniform(i, np), part = i - k * np, sub = BM < DS_GEMM_BM ? part & 1 : 0, n0 = (BM < DS_GEMM_BM ? part >> 1 : part) * BN;
    const int slot0 = __builtin_amdgcn_readlane(o0, q), rows_g = (__builtin_amdgcn_readlane(o1, q) - slot0) * rows;
    const int g0 = (8 * (__builtin_amdgcn_readlane(k0, q) + k) + die - __builtin_amdgcn_readlane(mend - nm, q)) * DS_GEMM_BM + sub * BM;
    if (g0 >= rows_g) return;
    const int k_in = __builtin_amdgcn_readlane(ki, q), k_out = __builtin_amdgcn_readlane(ko, q), row = lanes.row(T - 1 - q);
    // (up to 64 filters left: two wavefronts side by side, so that none is without)
    if constexpr (BM == 128) {
        if (k_out - n0 > 64) body<S, 4, 4, 9, 3>(a, t, g0, slot0, rows_g, n0, k_in, k_out, row, smem);
        else body<S, 2, 2, 9, 3>(a, t, g0, slot0, rows_g, n0, k_in, k_out, row, smem);
    } else {
        if (k_out - n0 > 64) body<S, 2, 4, 18, 3>(a, t, g0, slot0, rows_g, n0, k_in, k_out, row, smem);
        else body<S, 1, 2, 18, 3>(a, t, g0, slot0, rows_g, n0, k_in, k_out, row, smem);
    }
}

template <int S, int BM>
int32_t launch(const GemmArgs& a, const Conv3T& t, int32_t max_mtiles, int32_t max_kout, hipStream_t s) {
    const int32_t rc = ds_reserve_lds((const void*)conv3_tiled_kernel<S, BM>, smem_bytes(S, BM), "sliced 3x3 conv on tiled filters");
    if (rc) return rc;
    const int die = (max_mtiles + 7) / 8 * (DS_GEMM_BM / BM) * ((max_kout + BN - 1) / BN);
    ProfScope prof(DS_K_CONV3, s);
    hipLaunchKernelGGL((conv3_tiled_kernel<S, BM>), dim3((unsigned)(8 * die)), dim3(256), smem_bytes(S, BM), s, a, t);
    DS_CHECK_LAUNCH("sliced 3x3 conv on tiled filters");
    return DS_OK;
}

}  // namespace

// tiles: filters [ceil(N / 32)][18 ceil(K / 32) + 1] tiles of 1 KiB; channels: K as stored.  Launches of up to 600 of gemm_small_kernel's 32 x 32 tiles
// stay there, with up to eight wavefronts on a tile's reduction: us a pass, there / here, DS-ResNet 1 / 4 / 8 / 16 / 24 images 352 / 459 / 516 / 594 / 646 and 389 / 501 / 543 / 604 /
// 644, DS-ResNet++ 4 / 8 / 16 images 430 / 505 / 579 and 469 / 532 / 589.  With all of its launches there (up to 1000 tiles) DS-ResNet 14 / 16 / 18 / 33 images 597 / 601 / 633 / 687, as
// it is 590 / 594 / 620 / 690; three networks in turn 636 / 642 / 676 / 766 and 645 / 650 / 680 / 773: there filters come from memory, and more wavefronts ask for them.
// (The reduction dealt to two groups of wavefronts here: 33 images of DS-ResNet++ in turn 849 where 838 without.)
// Tiles of 64 pixels until there are enough of 128 to go round, us a pass, the line at 500 / 700 / 1200 / 1700 workgroups of 128 x 64: DS-ResNet 96 images 1164 / 1156 / 1156 / 1156, 128
// images 1401 / 1395 / 1403 / 1403, 160 images 1616 / 1609 / 1629 / 1629, 192 images 1860 / 1860 / 1856 / 1880, 256 images 2328 / 2327 / 2336 / 2359, in four parts 2317 / 2318 / 2315 / 2302.
// Stride 2, where gemm_kernel gathers the input of each tap again: us a launch, there / here, 256 images, 256 filters 50 / 46, 512 filters 56 / 45, 33 images of
// DS-ResNet++, 128 / 256 / 512 filters 22 / 17, 25 (gemm_small_kernel) / 16, 27 (the same) / 26.  Up to 128 filters gemm_kernel reads the input once as well and here 64 pixels of it feed
// one column tile only, so from 768 row tiles on it stays there: a launch of 128 / 160 / 256 images 40 / 51 / 70 and 38 / 45 / 72.  us a pass,
// there / here: DS-ResNet 128 images (799 row tiles) 1395 / 1394, 144 (898) 1504 / 1500, 160 (996) 1609 / 1603, 192 (1191) 1860 / 1858, 224 (1387) 2086 / 2089, 256 (1583) 2327 / 2330, in four
// parts 2318 / 2326, on uneven routes 2269 / 2277; DS-ResNet++ 128 images 1547 / 1544, 192 2089 / 2089, 256 2637 / 2640.  (Up to 1200 row tiles either is as good to 0.4 %, beyond
// them gemm_kernel by as much.)
int32_t ds_launch_conv3_tiled(const GemmArgs& a, const bf16_t* tiles, int32_t channels, int32_t max_mtiles, int32_t max_kout, hipStream_t s) {
    if (a.K != 3 || a.Kw > 3 || (a.stride != 1 && a.stride != 2) || a.stride_w > 0 || a.pad != 1 || a.n_seg != 1 || a.Ho != (a.H - 1) / a.stride + 1 ||
        a.Wo != (a.W - 1) / a.stride + 1 || a.rows != a.Ho * a.Wo || a.R || !conv_result(a) || !a.offsets)
        return DS_EUNSUPPORTED;
    // quotients in fp32, byte offsets of 31 bits
    if (a.B <= 0 || (int64_t)a.B * (a.H + 1) * (a.W + 3) >= 1 << 21 || (int64_t)a.B * a.a_sample_stride * 2 >= 0x7fffffffLL) return DS_EUNSUPPORTED;
    if (a.stride == 1 ? !conv3_fits(128, a.W, a.H) || !conv3_fits(64, a.W, a.H) : !conv3_fits2(a.W, a.H)) return DS_EUNSUPPORTED;
    const int64_t small = (int64_t)a.B * a.rows / 32 * ((max_kout + 31) / 32);
    if (small <= 600 && ds_gemm_small_takes(a, max_mtiles, max_kout)) return DS_EUNSUPPORTED;
    const Conv3T t = {tiles, (channels + 31) / 32 * CHUNK + 1};
    const int64_t crowd = a.crowd > 1 ? a.crowd : 1;
    if (a.stride == 2 && max_kout <= BN && max_mtiles * crowd >= 768) return DS_EUNSUPPORTED;
    if (a.stride == 2) return launch<2, 64>(a, t, max_mtiles, max_kout, s);
    const int64_t wgs = (int64_t)max_mtiles * ((max_kout + 63) / 64) * crowd;
    return wgs > 700 ? launch<1, 128>(a, t, max_mtiles, max_kout, s) : launch<1, 64>(a, t, max_mtiles, max_kout, s);
}
