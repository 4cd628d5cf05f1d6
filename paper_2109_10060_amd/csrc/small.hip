// Grouped prefix-slice GEMM / implicit-GEMM convolution for launches too small for the 128-row tile.
//
// With one to a few dozen samples a layer has 49 to a few thousand rows: gemm_kernel's 128 x 64 tiles then leave most of
// the 256 compute units without a workgroup, and the workgroups that exist walk the whole reduction alone (one image,
// last ResNet stage: 8 workgroups, up to 36 dependent 128-deep slabs).  What bounds such a launch is
// the length of that chain, so here the reduction is cut as well: a wavefront owns a WM*32 x WN*32 tile and every KS-th
// 64-deep slab of its reduction, the KS partial tiles are added in LDS in wavefront order, and a wavefront keeps PD
// slabs travelling in registers.  Its operand slabs go through an LDS region of its own (global loads cover whole
// 128-byte lines, the matrix operands want one row per lane), so there is no workgroup barrier before the final sum.
// Around that chain lie the round trips of the kernel's head and tail, and instructions: eight wavefronts of a compute unit
// issue one each in eight clocks.  So all kernel arguments are read at once, with the group table beside the tile record, the
// batch-norm rows and the residual are asked for behind the first operands, and a tap costs two instructions a row: a mask of
// the filter rows and columns inside the map, the pixel of a tap in the load's scalar offset.  One image of DS-ResNet, 52
// of these launches (44 and 4 pairs since): 431 -> 385 us a pass.
// Same tile list, row addressing, slices and epilogue as gemm_kernel; a list tile of 128 rows is walked in parts of
// WM*32 rows and a part beyond the group's rows ends at once.
// Column tiles are the fastest index of the launch: neighbouring workgroups land on different dies, so a die's L2 holds
// an eighth of the weights, which are most of what such a launch reads.
#include "tile_out.h"

namespace {

constexpr uint32_t OOB = 0x80000000u;

// 16-byte chunk c of a 128-byte LDS row r is stored at chunk position c ^ key(r): the row-major stores (8 lanes a row)
// and the operand reads (32 consecutive rows, one chunk column) are free of bank conflicts
__device__ __forceinline__ int key(int r) { return (r ^ (r >> 3)) & 7; }

// NW wavefronts: KS shares of the reduction x NW / KS column tiles
template <int WM, int WN, int NW, int KS, int PD, bool CONV, bool HASR>
__device__ __forceinline__ void small_tile(const GemmArgs& a, char* smem, int y, const int mi) {
    constexpr int BM = WM * 32, WBN = WN * 32, NC = NW / KS, BN = NC * WBN, BK = 64;
    constexpr int NSUB = DS_GEMM_BM / BM;
    constexpr int NA = BM / 8, NB = WBN / 8;                  // 16-byte loads of a lane per slab
    constexpr int WAVE_BYTES = (BM + WBN) * BK * 2;
    constexpr int ST_LD = WBN + 4;                            // staging: one fp32 tile per wavefront
    constexpr int STAGE_BYTES = BM * ST_LD * 4;
    constexpr int PER_WAVE = WAVE_BYTES > STAGE_BYTES ? WAVE_BYTES : STAGE_BYTES;

    const int mt = mi / NSUB, sub = mi - mt * NSUB;
    const GroupLanes lanes(a.gt);
    const bf16_t *A = a.A, *Wt = a.Wt, *R = a.R;
    void* C = a.C;
    const float *scale = a.scale, *shift = a.shift;
    const int32_t *a_index = a.a_index, *c_index = a.c_index;
    int64_t a_ss = a.a_sample_stride, c_ss = a.c_sample_stride, r_ss = a.r_sample_stride, c_segs = a.c_seg_stride;
    int a_ld = a.a_ld, c_ld = a.c_ld, r_ld = a.r_ld, c_row0 = a.c_row0, r_use = a.r_use_index;
    int w_ld = (int)a.w_ld, w_tap = (int)a.w_tap_stride, w_seg = (int)a.w_seg_stride;      // (in reach of 32 bits: ds_launch_gemm_small)
    int n_seg = a.n_seg, tab_ld = a.tab_ld, tab_seg = a.tab_seg_stride, rows = a.rows, act = a.act, out_f32 = a.out_f32;
    int H = a.H, W = a.W, Wo = a.Wo, KH = a.K, KW = a.Kw, sy = a.stride, sx = a.stride_w, pad = a.pad;
    const int4 me = ds_tile_record(a, mt);
    ds_hold(A, Wt, R, C, scale, shift, a_index, c_index, a_ss, c_ss, r_ss, c_segs, a_ld, c_ld, r_ld, c_row0, r_use, w_ld, w_tap,
            w_seg, n_seg, tab_ld, tab_seg, rows, act, out_f32);
    if constexpr (CONV) ds_hold(H, W, Wo, KH, KW, sy, sx, pad);
    if (me.x < 0) return;
    const int g = me.x, grow0 = me.y + sub * BM, slot0 = me.z, rows_g = me.w;
    if (grow0 >= rows_g) return;
    const int k_in = lanes.k_in(g), k_out = lanes.k_out(g);
    if (k_in <= 0 || k_out <= 0) return;
    int seg = 0;
    if (n_seg > 1) {
        const int ntiles = (k_out + BN - 1) / BN;
        seg = y / ntiles;
        if (seg >= n_seg) return;
        y -= seg * ntiles;
    }
    const int n0 = y * BN;
    if (n0 >= k_out) return;

    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, l32 = lane & 31, lhi = lane >> 5;
    const int ks = wave % KS, wc = wave / KS;                 // share of the reduction, column tile
    const int nw0 = n0 + wc * WBN;
    if (a_ld <= 0) a_ld = k_in;
    if (c_ld <= 0) c_ld = k_out;
    if (r_ld <= 0) r_ld = k_out;
    if (KW <= 0) KW = KH;
    if (sx <= 0) sx = sy;
    // A convolution's pixel offsets count from the first pixel that a filter at the map's corner covers, so that none is negative;
    // the descriptor starts there (what lies ahead of the map is never asked for).
    const int corner = CONV ? (pad * W + pad) * a_ld : 0;
    const __amdgpu_buffer_rsrc_t rsrc_a = __builtin_amdgcn_make_buffer_rsrc((void*)(A - corner), 0, 0x7fffffff, 0x00020000);
    const __amdgpu_buffer_rsrc_t rsrc_w = __builtin_amdgcn_make_buffer_rsrc((void*)Wt, 0, 0x7fffffff, 0x00020000);

    // ---- rows: lane r works out row r of the tile, the lanes that load it fetch the result from lane r
    uint32_t my_a = OOB;
    int my_taps = 0;                                          // filter rows (low half) and columns (high half) inside the map
    long long rc = -1, rr = 0;                                // output row (-1: no such row), residual row
    if (lane < BM) {
        const int m = grow0 + lane;
        if (m < rows_g) {
            const int sl = ds_quotient(m, rows), p = m - sl * rows, slot = slot0 + sl;
            const int sa = a_index ? a_index[slot] : slot;
            const int cs = c_index ? c_index[slot] : slot;
            int pix = p;
            if constexpr (CONV) {
                const int oy = ds_quotient(p, Wo), ox = p - oy * Wo;
                const int iy = oy * sy, ix = ox * sx;         // counted from the corner
                auto inside = [&](int i, int n, int k) {      // taps t < k with pad <= i + t < pad + n
                    const int lo = pad - i > 0 ? pad - i : 0, hi = pad + n - i < k ? pad + n - i : k;
                    return hi > lo ? (1 << hi) - (1 << lo) : 0;
                };
                my_taps = inside(iy, H, KH) | inside(ix, W, KW) << 16;
                pix = iy * W + ix;
            }
            my_a = (uint32_t)(((long long)sa * a_ss + (long long)pix * a_ld) * 2);
            const long long pc = p + c_row0;
            rc = (long long)cs * c_ss + pc * c_ld + (long long)seg * c_segs;
            rr = (long long)(r_use ? cs : 0) * r_ss + pc * r_ld;
        }
    }
    const int lrow = lane >> 3, lchunk = lane & 7, kc8 = lchunk * 8;
    uint32_t aoff[NA], woff[NB];
    int ataps[CONV ? NA : 1];
#pragma unroll
    for (int i = 0; i < NA; ++i) {
        aoff[i] = (uint32_t)__shfl((int)my_a, lrow + 8 * i, 64) + kc8 * 2;      // (no row: still out of range)
        if constexpr (CONV) ataps[i] = __shfl(my_taps, lrow + 8 * i, 64);
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int n = nw0 + lrow + 8 * i;
        woff[i] = n < k_out ? (uint32_t)(seg * w_seg + n * w_ld + kc8) * 2 : OOB;
    }

    const int kchunks = (k_in + BK - 1) / BK;
    const int nk = CONV ? KH * KW * kchunks : kchunks;
    uint4 ra[PD][NA], rb[PD][NB];
    // slab being fetched next: tap (row u, column v) and 64-channel chunk (this wavefront takes every KS-th slab)
    int lkc = ks, lu = 0, lv = 0;
    auto fetch = [&](uint4 (&va)[NA], uint4 (&vb)[NB]) {
        if constexpr (CONV)
            while (lkc >= kchunks) {
                lkc -= kchunks;
                if (++lv == KW) lv = 0, ++lu;
            }
        const bool kok = lkc * BK + kc8 < k_in;
        const int soff_a = ((lu * W + lv) * a_ld + lkc * BK) * 2;
        const int soff_w = ((lu * KW + lv) * w_tap + lkc * BK) * 2;
        const int tap = 1 << lu | 0x10000 << lv;
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            const bool ok = CONV ? kok && (ataps[CONV ? i : 0] & tap) == tap : kok;
            const auto t = __builtin_amdgcn_raw_buffer_load_b128(rsrc_a, (int)(ok ? aoff[i] : OOB), soff_a, 0);
            va[i] = make_uint4(t[0], t[1], t[2], t[3]);
        }
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const auto t = __builtin_amdgcn_raw_buffer_load_b128(rsrc_w, (int)(kok ? woff[i] : OOB), soff_w, 0);
            vb[i] = make_uint4(t[0], t[1], t[2], t[3]);
        }
        lkc += KS;
    };
#pragma unroll
    for (int st = 0; st < PD; ++st)
        if (ks + KS * st < nk) fetch(ra[st], rb[st]);

    // What the epilogue adds is requested behind the first operands: a thread finishes 4 channels, the same for all of its
    // rows.  Asked for after the final sum it was one more round trip to memory in a launch that is a chain of four.
    constexpr int GPR = BN / 4, RSTEP = 64 * NW / GPR, NE = (BM + RSTEP - 1) / RSTEP;
    const int er0 = tid / GPR, c4 = (tid - er0 * GPR) * 4, n = n0 + c4;
    float vs[4] = {1.f, 1.f, 1.f, 1.f}, vh[4] = {0.f, 0.f, 0.f, 0.f};
    long long coff[NE];
    uint2 res[HASR ? NE : 1];
    if (n < k_out) {
        const long long ti = (long long)lanes.row(g) * tab_ld + (long long)seg * tab_seg + n;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            if (scale) vs[q] = scale[ti + q];
            if (shift) vh[q] = shift[ti + q];
        }
    }
#pragma unroll
    for (int i = 0; i < NE; ++i) {
        const int r = er0 + i * RSTEP;                        // (lanes past the tile read some lane's row and drop it)
        const long long c = __shfl(rc, r & 63, 64), ro = __shfl(rr, r & 63, 64);
        coff[i] = r < BM && n < k_out ? c : -1;
        if constexpr (HASR) {
            res[i] = make_uint2(0, 0);
            if (coff[i] >= 0) res[i] = *(const uint2*)(R + ro + n);
        }
    }

    f32x16_t acc[WM][WN];
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int j = 0; j < WN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

    // LDS written and read by one wavefront: its accesses complete in order, only the compiler has to be kept in line
    bf16_t* As = (bf16_t*)(smem + wave * PER_WAVE);
    bf16_t* Bs = As + BM * BK;
    auto stage = [&](const uint4 (&va)[NA], const uint4 (&vb)[NB]) {
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            const int r = lrow + 8 * i;
            *(uint4*)(As + r * BK + ((lchunk ^ key(r)) * 8)) = va[i];
        }
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const int r = lrow + 8 * i;
            *(uint4*)(Bs + r * BK + ((lchunk ^ key(r)) * 8)) = vb[i];
        }
        wave_sync();
    };
    bf16x8_t af[BK / 16][WM], bf[BK / 16][WN];
    auto operands = [&]() {
#pragma unroll
        for (int kk = 0; kk < BK / 16; ++kk) {
            const int c = kk * 2 + lhi;
#pragma unroll
            for (int t = 0; t < WM; ++t) af[kk][t] = *(const bf16x8_t*)(As + (t * 32 + l32) * BK + ((c ^ key(t * 32 + l32)) * 8));
#pragma unroll
            for (int t = 0; t < WN; ++t) bf[kk][t] = *(const bf16x8_t*)(Bs + (t * 32 + l32) * BK + ((c ^ key(t * 32 + l32)) * 8));
        }
        wave_sync();
    };
    for (int base = ks; base < nk; base += KS * PD) {
#pragma unroll
        for (int st = 0; st < PD; ++st) {
            const int kt = base + KS * st;
            if (kt >= nk) break;                              // uniform over the wavefront
            stage(ra[st], rb[st]);
            if (kt + KS * PD < nk) fetch(ra[st], rb[st]);
            operands();
#pragma unroll
            for (int kk = 0; kk < BK / 16; ++kk)
#pragma unroll
                for (int i = 0; i < WM; ++i)
#pragma unroll
                    for (int j = 0; j < WN; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[kk][i], bf[kk][j], acc[i][j], 0, 0, 0);
        }
    }

    // ---- partial tiles to LDS, summed in wavefront order; a lane finishes 4 consecutive channels of one row
    float* st = (float*)(smem + wave * PER_WAVE);
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int j = 0; j < WN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v)
                st[(i * 32 + 8 * (v >> 2) + 4 * lhi + (v & 3)) * ST_LD + j * 32 + l32] = acc[i][j][v];
    __syncthreads();
    const int ct = c4 / WBN, cl = c4 - ct * WBN;
    auto finish = [&](auto gelu) __attribute__((always_inline)) {
        constexpr bool GELU = decltype(gelu)::value;
#pragma unroll
        for (int i = 0; i < NE; ++i) {
            if (coff[i] < 0) continue;
            const int r = er0 + i * RSTEP;
            float val[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int w = 0; w < KS; ++w) {
                const float4 t = *(const float4*)((const float*)(smem + (ct * KS + w) * PER_WAVE) + r * ST_LD + cl);
                val[0] += t.x; val[1] += t.y; val[2] += t.z; val[3] += t.w;
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) val[q] = val[q] * vs[q] + vh[q];
            if constexpr (HASR) {
                val[0] += __uint_as_float(res[i].x << 16);
                val[1] += __uint_as_float(res[i].x & 0xffff0000u);
                val[2] += __uint_as_float(res[i].y << 16);
                val[3] += __uint_as_float(res[i].y & 0xffff0000u);
            }
            if (GELU ? out_f32 : act == DS_ACT_RELU) {
#pragma unroll
                for (int q = 0; q < 4; ++q) val[q] = GELU ? gelu_erf(val[q]) : fmaxf(val[q], 0.f);
            }
            if (out_f32) *(float4*)((float*)C + coff[i] + n) = make_float4(val[0], val[1], val[2], val[3]);
            else if constexpr (GELU) *(uint2*)((bf16_t*)C + coff[i] + n) = gelu_bf16x4(val[0], val[1], val[2], val[3]);
            else *(uint2*)((bf16_t*)C + coff[i] + n) = make_uint2(f2bf2(val[0], val[1]), f2bf2(val[2], val[3]));
        }
    };
    // (each in code of its own: with that of GELU between the others one image of DS-ResNet took 358 us, 352 here)
    if (act == DS_ACT_GELU) finish(std::true_type());
    else finish(std::false_type());
}

template <int WM, int WN, int NW, int KS, int PD, bool CONV, bool HASR>
__global__ __launch_bounds__(64 * NW) void gemm_small_kernel(const GemmArgs a) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    small_tile<WM, WN, NW, KS, PD, CONV, HASR>(a, smem, (int)blockIdx.x, (int)blockIdx.y);
}

// two launches that do not wait for one another as one: the workgroups [0, split) are those of p[0], the others those of p[1], each
// with its own number of column tiles (on a grid as wide as the wider one, the workgroups that only end cost more than the launch:
// one image of DS-ResNet 371 -> 385 us a pass)
struct SmallPair {
    GemmArgs p[2];
    int32_t split, ny[2];
};

template <int WM, int WN, int NW, int KS, int PD, bool CONV>
__global__ __launch_bounds__(64 * NW) void gemm_small_pair_kernel(const SmallPair a) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const unsigned second = (int)blockIdx.x >= a.split, i = blockIdx.x - (second ? a.split : 0), ny = second ? a.ny[1] : a.ny[0], mi = i / ny;
    small_tile<WM, WN, NW, KS, PD, CONV, false>(a.p[second], smem, (int)(i - mi * ny), (int)mi);
}

template <int WM, int WN, int NW, int KS>
struct SmallTile {
    static constexpr int BM = WM * 32, WBN = WN * 32, BN = (NW / KS) * WBN;
    static constexpr int W1 = (BM + WBN) * 128, W2 = BM * (WBN + 4) * 4;
    static constexpr int SMEM = NW * (W1 > W2 ? W1 : W2);
};

template <int WM, int WN, int NW, int KS, int PD, bool CONV>
int32_t launch_pair(SmallPair& a, int32_t tiles0, int32_t kout0, int32_t tiles1, int32_t kout1, hipStream_t s) {
    using K = SmallTile<WM, WN, NW, KS>;
    auto kern = gemm_small_pair_kernel<WM, WN, NW, KS, PD, CONV>;
    const int32_t rc = ds_reserve_lds((const void*)kern, K::SMEM, "pair of small sliced gemms");
    if (rc) return rc;
    a.ny[0] = (kout0 + K::BN - 1) / K::BN;
    a.ny[1] = (kout1 + K::BN - 1) / K::BN;
    a.split = tiles0 * (DS_GEMM_BM / K::BM) * a.ny[0];
    ProfScope prof(DS_K_SMALL, s);
    hipLaunchKernelGGL(kern, dim3((unsigned)(a.split + tiles1 * (DS_GEMM_BM / K::BM) * a.ny[1])), dim3(64 * NW), K::SMEM, s, a);
    DS_CHECK_LAUNCH("pair of small sliced gemms");
    return DS_OK;
}

template <int WM, int WN, int NW, int KS, int PD, bool CONV, bool HASR>
int32_t launch(const GemmArgs& a, int32_t max_mtiles, int32_t max_kout, hipStream_t s) {
    using K = SmallTile<WM, WN, NW, KS>;
    constexpr int BM = K::BM, BN = K::BN, SMEM = K::SMEM;
    auto kern = gemm_small_kernel<WM, WN, NW, KS, PD, CONV, HASR>;
    const int32_t rc = ds_reserve_lds((const void*)kern, SMEM, "small sliced gemm");
    if (rc) return rc;
    const int ny = a.n_seg * ((max_kout + BN - 1) / BN);
    ProfScope prof(DS_K_SMALL, s);
    hipLaunchKernelGGL(kern, dim3((unsigned)ny, (unsigned)(max_mtiles * (DS_GEMM_BM / BM))), dim3(64 * NW), SMEM, s, a);
    DS_CHECK_LAUNCH("small sliced gemm");
    return DS_OK;
}

// 32 x 32 tiles a launch can have and 64-deep slabs of its reduction
struct SmallSize {
    int kmax, taps, nk;
    long long t;
};
SmallSize small_size(const GemmArgs& a, int32_t max_kout) {
    SmallSize z;
    z.kmax = 0;
    for (int t = 0; t < a.gt.T; ++t) z.kmax = a.gt.k_in[t] > z.kmax ? a.gt.k_in[t] : z.kmax;
    z.taps = a.K * (a.Kw > 0 ? a.Kw : a.K);
    z.nk = z.taps * ((z.kmax + 63) / 64);
    const long long groups = a.B < a.gt.T ? a.B : a.gt.T, rows = (long long)a.B * a.rows;
    z.t = ((rows - groups) / 32 + groups) * a.n_seg * ((max_kout + 31) / 32);
    return z;
}
int small_choice(long long t, int nk) {
    if (t <= 340 && nk > 2) return 0;
    if (t > 340 && t <= 500 && nk >= 5) return 1;
    if (t <= 700) return 2;
    return nk >= 24 ? 3 : nk > 4 ? 4 : 5;
}
// 32-bit byte offsets inside the kernel
bool small_in_reach(const GemmArgs& a, const SmallSize& z, int32_t max_mtiles, int32_t max_kout) {
    const long long slots = (long long)max_mtiles * DS_GEMM_BM / (a.rows > 0 ? a.rows : 1) + 1;
    const long long corner = (long long)a.pad * (a.W + 1) * (a.a_ld > z.kmax ? a.a_ld : z.kmax);
    if ((slots * a.a_sample_stride + corner) * 2 >= 0x7fffffffLL) return false;
    return ((long long)a.n_seg * a.w_seg_stride + (long long)max_kout * a.w_ld + z.taps * a.w_tap_stride + z.kmax) * 2 < 0x7fffffffLL;
}

}  // namespace

// Which tile, by the number t of 32 x 32 tiles the launch can have and the number nk of 64-deep slabs of its reduction.
// Measured on the layers of DS-ResNet with the benchmark's routes, kernel time in us, general kernels -> here
// (profiles/dispatch_choices.txt; stages counted from 1):
//   t <= 340    one tile and 8 shares of the reduction per workgroup: every compute unit gets at most one or two, so the
//               length of a share is all that counts (stage 4, one sample: 3x3 8.9 -> 5.7, first 1x1 6.9 -> 4.4; four samples
//               22.9 -> 11.0, 16.0 -> 7.8)
//   t <= 500    32 x 64 tiles, 8 shares (stage 3, eight samples: 3x3 15.7 -> 10.7, 1x1 11.3 -> 8.0), 32 x 32 and 4 shares
//               when there are fewer slabs than shares (stage 4, four samples, last 1x1 8.1 -> 6.2)
//   t <= 700    32 x 32, 4 shares (stage 4, 16 samples: 1x1 17.0 -> 9.4, 3x3 23.8 -> 14.0)
//   t <= 1000   64 x 64 tiles, 8 shares, for 24 slabs and more (stage 3, 16 samples: 3x3 15.2 -> 12.6), 32 x 64 tiles and 4
//               shares (1x1 11.6 -> 9.3; stage 1, four samples: 3x3 8.3 -> 9.4, the one measured layer that loses), two column tiles and 2 shares
//               up to four slabs (stage 3, four samples, last 1x1 7.8 -> 6.6)
//   ordered     one wavefront walks a tile's whole reduction, three slabs ahead, two tiles per workgroup, up to 1700 tiles
//               (patch embedding of DS-ViT, twelve slabs, 1 / 5 / 16 images 13.6 -> 9.3 / 15.6 -> 10.5 / 14.6 -> 10.5)
//   beyond      the 128-row kernels have enough workgroups and read less per product -- except the strided KxK layers
//               (no staged patch for them), which stay here up to 1700 tiles (stage 4, 33 samples 34.3 -> 20.1)
bool ds_gemm_small_takes(const GemmArgs& a, int32_t max_mtiles, int32_t max_kout) {
    if (max_mtiles <= 0 || max_kout <= 0 || a.B <= 0) return false;
    if (a.K > 15 || a.Kw > 15) return false;                  // tap masks of 16 bits
    const SmallSize z = small_size(a, max_kout);
    const bool strided = z.taps > 1 && a.stride > 1;
    if (z.t > 1700 || (z.t > 1000 && !a.ordered && !(strided && z.nk >= 24))) return false;
    return small_in_reach(a, z, max_mtiles, max_kout);
}

int32_t ds_launch_gemm_small(const GemmArgs& a, int32_t max_mtiles, int32_t max_kout, hipStream_t s) {
    if (!ds_gemm_small_takes(a, max_mtiles, max_kout)) return DS_EUNSUPPORTED;
    const bool conv = a.K > 1 || a.stride > 1 || a.pad > 0;
    const SmallSize z = small_size(a, max_kout);
    const int nk = z.nk;
    const long long t = z.t;
#define DS_SMALL(...)                                                                       \
    (conv ? (a.R ? launch<__VA_ARGS__, true, true>(a, max_mtiles, max_kout, s)               \
                 : launch<__VA_ARGS__, true, false>(a, max_mtiles, max_kout, s))             \
          : (a.R ? launch<__VA_ARGS__, false, true>(a, max_mtiles, max_kout, s)              \
                 : launch<__VA_ARGS__, false, false>(a, max_mtiles, max_kout, s)))
    if (a.ordered) return DS_SMALL(1, 1, 2, 1, 3);
    switch (small_choice(t, nk)) {
        case 0: return DS_SMALL(1, 1, 8, 8, 4);
        case 1: return DS_SMALL(1, 2, 8, 8, 2);
        case 2: return DS_SMALL(1, 1, 4, 4, 4);
        case 3: return DS_SMALL(2, 2, 8, 8, 1);
        case 4: return DS_SMALL(1, 2, 4, 4, 2);
        default: return DS_SMALL(1, 1, 4, 2, 4);
    }
#undef DS_SMALL
}

// A stage's projection and first layer both read its input and one waits for neither; with a few samples each is mostly the 4 to 6 us
// of a launch that has one before it.  Paired where the two have as many tiles together as one launch here may have.  DS-ResNet,
// two launches -> here: 1 image 370 -> 362 us a pass, 2 / 4 / 8 images 437.6 / 509.5 / 596.7 -> 436.5 / 507.8 / 594.1 (fewer stages
// pair); DS-ResNet++ 1 image 311 -> 299.5.
int32_t ds_launch_gemm_small_pair(const GemmArgs& a, int32_t mtiles_a, int32_t kout_a, const GemmArgs& b, int32_t mtiles_b, int32_t kout_b,
                                  hipStream_t s) {
    if (mtiles_a <= 0 || mtiles_b <= 0 || kout_a <= 0 || kout_b <= 0 || a.B <= 0 || b.B <= 0) return DS_EUNSUPPORTED;
    // 1x1 layers without residual and segments
    for (const GemmArgs* p : {&a, &b})
        if (p->K != 1 || p->Kw > 1 || p->pad || p->R || p->ordered || p->n_seg != 1) return DS_EUNSUPPORTED;
    const SmallSize za = small_size(a, kout_a), zb = small_size(b, kout_b);
    if (za.t + zb.t > 1000 || !small_in_reach(a, za, mtiles_a, kout_a) || !small_in_reach(b, zb, mtiles_b, kout_b)) return DS_EUNSUPPORTED;
    SmallPair p;
    p.p[0] = a; p.p[1] = b;
    const bool conv = a.stride > 1 || b.stride > 1;
    // The tile that either layer takes alone, so that pairing changes no sum; one slab is summed the same way in every tile.
    const int ca = small_choice(za.t, za.nk), cb = small_choice(zb.t, zb.nk);
    if (ca != cb && (za.nk > 1 || zb.nk > 1)) return DS_EUNSUPPORTED;
#define DS_PAIR(...) (conv ? launch_pair<__VA_ARGS__, true>(p, mtiles_a, kout_a, mtiles_b, kout_b, s) : launch_pair<__VA_ARGS__, false>(p, mtiles_a, kout_a, mtiles_b, kout_b, s))
    switch (za.t > zb.t ? ca : cb) {
        case 0: return DS_PAIR(1, 1, 8, 8, 4);
        case 1: return DS_PAIR(1, 2, 8, 8, 2);
        case 2: return DS_PAIR(1, 1, 4, 4, 4);
        case 4: return DS_PAIR(1, 2, 4, 4, 2);
        case 5: return DS_PAIR(1, 1, 4, 2, 4);
        default: return DS_EUNSUPPORTED;
    }
#undef DS_PAIR
}
