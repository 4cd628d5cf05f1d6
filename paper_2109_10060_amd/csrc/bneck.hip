// The rest of a bottleneck block behind its first layer, in one kernel (filter slicing, Section 3.3 Eq. 9; split batch-norm, Eq. 14):
//   y2 = relu(bn(conv3x3(y1)));  z = relu(bn(conv1x1(y2)) + shortcut);  next y1 = relu(bn(conv1x1(z)))
// for every route group, stride 1, slices of at most 32 NB mid channels.  The shortcut is read (z may be updated in place) or, with
// PROJ, computed from the stage's input; the next block's first layer rides along with CHAIN.
//
// What bounds it: these stages are streams (the wide maps in and out), and as separate launches the 3x3 layer is mostly the
// head and the epilogue of its workgroups -- tile record, row tables, first slab, staging -- around a few matrix instructions.  Here a
// workgroup of four wavefronts owns 128 pixels from the 3x3 layer to the next block's input.  conv3_kernel's patch scheme first; its
// results never reach LDS: a lane holds four consecutive channels of its own pixel, and v_permlane32_swap between the two halves
// of a wavefront makes them the operand of the next product.  Then thin_kernel's passes of 64 output columns, what a pass needs
// (weights, shortcut rows) requested one pass ahead; a wavefront's rows of the shortcut and of the result are its own, so that
// only the weights need barriers.
//
// Measured, 256 images of DS-ResNet, us: first stage's first block (projection 78, 3x3 72, last and next first layer 131: together 281)
// 161, second (72 + 131) 156 at 4.5 TB/s, third (72 + 108) 132 with the sums for the next gate, 127 without; second stage's blocks (50 + 88) 112 and
// (50 + 66) 90 (profiles/layers_resnet_b256.txt).  Tried: weight slabs in turn
// with one barrier a pass and a phase (same time), tiles in plain order (1 % slower), two workgroups a compute unit in place of three
// with the projection inside (207 for 170), 32 columns of a pass after the other (1 % slower).
//
// Sums run in the order of conv3_kernel and thin_kernel where those do not deal a reduction to shares, and intermediate maps are rounded to
// bf16 as they would be in memory, so the results are the same bits as theirs.  Launches of few samples they do deal (conv3_kernel up
// to 512 workgroups, gemm_small_kernel), so there a batch of 2 to 20 images gets other last bits here than from the separate launches: the
// ones it gets in a batch of 33 (logits of DS-ResNet in batches of 5 against one of 256, 2-norm 8.7e-4 before and 7.8e-4 here).
#include "common.h"
#include <type_traits>

namespace {

constexpr int BM = DS_GEMM_BM, NT = 256, SUM_ROWS = DS_BNECK_SUM_ROWS;
constexpr uint32_t OOB = 0x80000000u;
static_assert(SUM_ROWS == 64 && BM == 2 * SUM_ROWS, "a half of the tile, two wavefronts, a piece of the sums");
constexpr int RMAX = 248, ZROW = RMAX;         // patch rows: 128 + 2 (W + 1), W <= 59; one more of zeros
constexpr int NR = (RMAX * 4 + NT - 1) / NT;
constexpr int TILE_BYTES = BM * 128;           // [128 rows][64 columns], 16-byte chunk c of row r at c ^ (r & 7)

template <int NB, bool PROJ, bool CHAIN>
struct Layout {
    static constexpr int PATCH = (RMAX + 1) * 64, TAPS = 3 * NB * 32 * 64, CONV = PATCH + TAPS;
    static constexpr int W3 = NB * 64 * 64, WP = PROJ ? 2 * 64 * 64 : 0, W1 = CHAIN ? 2 * NB * 32 * 64 : 0, SLAB = W3 + WP + W1;
    static constexpr int OUT = TILE_BYTES + SLAB;
    static constexpr int MAIN = CONV > OUT ? CONV : OUT;
    static constexpr int N_OUT = 128 * NB;                      // output columns the constants have room for
    static constexpr int CST = MAIN, ROWS = CST + (PROJ ? 4 : 2) * N_OUT * 4, CST2 = ROWS + 2 * BM * 4, SUMS = CST2 + (CHAIN ? 4 : 2) * NB * 32 * 4;
    // without a next block: column sums of each wavefront's rows
    static constexpr int SMEM = SUMS, SMEM_SUMS = SUMS + 4 * N_OUT * 4;
};

__device__ __forceinline__ int sw(int r) { return ((r >> 1) ^ (r >> 2)) & 3; }
__device__ __forceinline__ uint4 load16(const __amdgpu_buffer_rsrc_t& rs, uint32_t off, int soff = 0) {
    const auto t = __builtin_amdgcn_raw_buffer_load_b128(rs, (int)off, soff, 0);
    return make_uint4(t[0], t[1], t[2], t[3]);
}
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
__device__ __forceinline__ void add_bf16x4(float (&v)[4], const uint2 r) {
    v[0] += __uint_as_float(r.x << 16);
    v[1] += __uint_as_float(r.x & 0xffff0000u);
    v[2] += __uint_as_float(r.y << 16);
    v[3] += __uint_as_float(r.y & 0xffff0000u);
}

// sum over the lanes 8, 16, 24, .. away, all of them get it: a rotation within 16 lanes, then rows and halves of the wavefront traded
__device__ __forceinline__ float sum_of_8(float v) {
    v += __uint_as_float(__builtin_amdgcn_update_dpp(0, __float_as_uint(v), 0x128, 0xf, 0xf, true));
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

template <int NB, bool PROJ, bool CHAIN>
__global__ __launch_bounds__(NT, NB == 2 ? 3 : 2) void bneck_kernel(const BneckArgs args, const int max_mtiles0) {
    using L = Layout<NB, PROJ, CHAIN>;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    char* As = smem;                                   // [RMAX + 1][32] bf16: the patch of a chunk
    char* Ts = smem + L::PATCH;                        // [3][32 NB][32] bf16: weights of a filter row
    char* tile = smem;                                 // after the 3x3 layer: shortcut in, result out
    float* cst = (float*)(smem + L::CST);              // scale, shift (PROJ: the projection's behind them) [N_OUT] each
    int* rowZ = (int*)(smem + L::ROWS);                // element offsets; < 0: no such row
    int* row1 = rowZ + BM;
    float* cst2 = (float*)(smem + L::CST2);            // [32 NB] scale, shift of the 3x3 layer; CHAIN: of the next block's first

    // Eight neighbouring tiles to a die (workgroups are dealt to the dies in turn): the patches of neighbours overlap by almost half.
    const int b = (int)blockIdx.x, mt = (b & ~63) | ((b & 7) << 3) | ((b >> 3) & 7);
    const GroupLanes lanes(args.gt);
    const int next_g = CHAIN ? args.next[threadIdx.x & 63] : 0, kx_g = PROJ ? args.kx[threadIdx.x & 63] : 0;
    struct {                                           // the arguments, asked for together (ds_hold)
        const bf16_t *y1, *w2, *w3, *w1, *wp, *shortcut, *x;
        const float *s2, *h2, *s3, *h3, *s1, *h1, *sp, *hp;
        const int32_t* x_index;
        bf16_t *z, *y1_next;
        float* sums;
        int64_t y1_ss, z_ss, x_ss;
        int mid_full, out_full, x_full, tab3, H, W;
        const int4* mtiles;
        const int32_t* n_mtiles;
    } a = {args.y1, args.w2, args.w3, args.w1, args.wp, args.shortcut, args.x, args.s2, args.h2, args.s3, args.h3, args.s1, args.h1, args.sp,
           args.hp, args.x_index, args.z, args.y1_next, args.sums, args.y1_ss, args.z_ss, args.x_ss, args.mid_full, args.out_full, args.x_full,
           args.tab3, args.H, args.W, args.mtiles, args.n_mtiles};
    int max_mtiles = max_mtiles0;
    ds_hold(max_mtiles, a.mtiles, a.n_mtiles, a.y1, a.w2, a.w3, a.s2, a.h2, a.s3, a.h3, a.z, a.y1_ss, a.z_ss, a.mid_full, a.tab3, a.H, a.W);
    if constexpr (CHAIN) ds_hold(a.w1, a.s1, a.h1, a.y1_next, a.out_full);
    else ds_hold(a.sums, a.out_full);
    if constexpr (PROJ) ds_hold(a.x, a.wp, a.sp, a.hp, a.x_index, a.x_ss, a.x_full);
    else ds_hold(a.shortcut);
    if (mt >= max_mtiles) return;
    const int4 me = a.mtiles[mt];
    const int n_mtiles = *a.n_mtiles;
    int first = __builtin_amdgcn_readfirstlane(me.x);
    ds_hold(first);                                    // asked for beside the count, not behind it
    if (mt >= n_mtiles) return;
    const int g = first, grow0 = me.y, slot0 = me.z, rows_g = me.w;
    const int mid = lanes.k_in(g), out = lanes.k_out(g), trow = lanes.row(g);
    if (mid <= 0 || out <= 0) return;
    const int W = a.W, H = a.H, rows = W * H, halo = W + 1, R = BM + 2 * halo;
    const int next = CHAIN ? __builtin_amdgcn_readlane(next_g, g) : 0;            // <= 0: this group ends with the block
    const int kx = PROJ ? __builtin_amdgcn_readlane(kx_g, g) : 0;

    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, l32 = lane & 31, lhi = lane >> 5;
    const __amdgpu_buffer_rsrc_t rs_y1 = __builtin_amdgcn_make_buffer_rsrc((void*)a.y1, 0, 0x7fffffff, 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_w2 = __builtin_amdgcn_make_buffer_rsrc((void*)a.w2, 0, 0x7fffffff, 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_w3 = __builtin_amdgcn_make_buffer_rsrc((void*)a.w3, 0, 0x7fffffff, 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_w1 = __builtin_amdgcn_make_buffer_rsrc((void*)(CHAIN ? a.w1 : a.w3), 0, 0x7fffffff, 0x00020000);
    const __amdgpu_buffer_rsrc_t rs_wp = __builtin_amdgcn_make_buffer_rsrc((void*)(PROJ ? a.wp : a.w3), 0, 0x7fffffff, 0x00020000);

    // ---- 3x3 layer: as conv3_kernel, filters as the row operand ---------------------------------------------------------------
    const int lchunk = tid & 3, wrow = tid >> 2;
    uint32_t poff[NR], woff[NB / 2];
    {
        // a wavefront loads 64 patch rows, 16 of every 64: a lane works out one of them, the lanes that load it get its address from there
        static_assert(NR == 4, "a patch row per lane");
        const int jr = 16 * wave + (lane & 15) + 64 * (lane >> 4), px = grow0 - halo + jr;
        uint32_t o = OOB;
        if (jr < R && px >= 0 && px < rows_g) {
            const int sl = ds_quotient(px, rows);
            o = (uint32_t)(((slot0 + sl) * a.y1_ss + (int64_t)(px - sl * rows) * mid) * 2);
        }
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            const uint32_t q = (uint32_t)__shfl((int)o, (lane >> 2) + 16 * i, 64);
            poff[i] = q == OOB ? OOB : q + lchunk * 16;
        }
    }
#pragma unroll
    for (int i = 0; i < NB / 2; ++i) woff[i] = wrow + 64 * i < mid ? (uint32_t)((wrow + 64 * i) * 9 * a.mid_full + lchunk * 8) * 2 : OOB;
    uint4 ra[NR], rb[3][NB / 2];
    auto load_phase = [&](int c, int u) __attribute__((always_inline)) {
        const bool kok = c * 32 + lchunk * 8 < mid;
        if (u == 0) {
#pragma unroll
            for (int i = 0; i < NR; ++i) ra[i] = load16(rs_y1, kok ? poff[i] : OOB, c * 64);
        }
#pragma unroll
        for (int v = 0; v < 3; ++v)
#pragma unroll
            for (int i = 0; i < NB / 2; ++i)
                rb[v][i] = load16(rs_w2, kok ? woff[i] : OOB, ((u * 3 + v) * a.mid_full + c * 32) * 2);
    };
    auto store_phase = [&](int u) __attribute__((always_inline)) {
        if (u == 0) {
#pragma unroll
            for (int i = 0; i < NR; ++i) {
                const int jr = (tid + NT * i) >> 2;
                if (jr < R) *(uint4*)(As + jr * 64 + ((lchunk ^ sw(jr)) * 16)) = ra[i];
            }
        }
#pragma unroll
        for (int v = 0; v < 3; ++v)
#pragma unroll
            for (int i = 0; i < NB / 2; ++i)
                *(uint4*)(Ts + (v * 32 * NB + wrow + 64 * i) * 64 + ((lchunk ^ sw(wrow)) * 16)) = rb[v][i];
    };
    load_phase(0, 0);
    if (tid < 4) *(uint4*)(As + ZROW * 64 + tid * 16) = make_uint4(0, 0, 0, 0);
    // ---- tables, worked out while the first loads travel ----------------------------------------------------------------------
    for (int i = tid; i < out; i += NT) {
        cst[i] = a.s3[(int64_t)trow * a.tab3 + i];
        cst[L::N_OUT + i] = a.h3[(int64_t)trow * a.tab3 + i];
        if constexpr (PROJ) {
            cst[2 * L::N_OUT + i] = a.sp[(int64_t)trow * a.tab3 + i];
            cst[3 * L::N_OUT + i] = a.hp[(int64_t)trow * a.tab3 + i];
        }
    }
    if (tid < mid) {
        cst2[tid] = a.s2[(int64_t)trow * a.mid_full + tid];
        cst2[32 * NB + tid] = a.h2[(int64_t)trow * a.mid_full + tid];
    }
    if (CHAIN && tid < next) {
        cst2[64 * NB + tid] = a.s1[(int64_t)trow * a.mid_full + tid];
        cst2[96 * NB + tid] = a.h1[(int64_t)trow * a.mid_full + tid];
    }
    const int prow = wave * 32 + l32;                  // this lane's pixel as an operand
    int tapmask = 0;
    uint32_t xoff = OOB;
    {
        const int m = grow0 + prow;
        int z = -1, y = -1;
        if (m < rows_g) {
            const int sl = ds_quotient(m, rows), p = m - sl * rows, slot = slot0 + sl;
            const int oy = ds_quotient(p, W), ox = p - oy * W;
            // filter columns, filter rows inside the map
            const int cols = (ox > 0 ? 1 : 0) | 2 | (ox + 1 < W ? 4 : 0);
            tapmask = (oy > 0 ? cols : 0) | cols << 3 | (oy + 1 < H ? cols << 6 : 0);
            z = (int)(slot * a.z_ss + (int64_t)p * out);
            y = (int)(slot * a.y1_ss + (int64_t)p * next);
            if constexpr (PROJ) {
                const int sx = a.x_index ? a.x_index[slot] : slot;
                xoff = (uint32_t)((sx * a.x_ss + (int64_t)p * kx + lhi * 8) * 2);
            }
        }
        if (lhi == 0) {
            rowZ[prow] = z;
            row1[prow] = y;
        }
    }

    f32x16_t acc[NB];
#pragma unroll
    for (int t = 0; t < NB; ++t)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[t][v] = 0.f;
    // the products of a phase with the filter blocks the slice has
    auto taps = [&](auto blocks, int u, int ksteps) __attribute__((always_inline)) {
        constexpr int N = decltype(blocks)::value;
#pragma unroll
        for (int v = 0; v < 3; ++v) {
            const int arow = ((tapmask >> (u * 3 + v)) & 1) ? prow + halo + (u - 1) * W + (v - 1) : ZROW;
            const char* ap = As + arow * 64;
            const int fa = sw(arow);
#pragma unroll
            for (int kk = 0; kk < 2; ++kk) {
                if (kk >= ksteps) continue;
                const int ch = kk * 2 + lhi;
                const bf16x8_t pf = *(const bf16x8_t*)(ap + ((ch ^ fa) * 16));
#pragma unroll
                for (int t = 0; t < N; ++t) {
                    const bf16x8_t wf = *(const bf16x8_t*)(Ts + (v * 32 * NB + t * 32 + l32) * 64 + ((ch ^ sw(l32)) * 16));
                    acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf, pf, acc[t], 0, 0, 0);
                }
            }
        }
    };

    // ---- what a pass of 64 output columns needs, one pass ahead ---------------------------------------------------------------
    constexpr int CP = NB * 4;                         // 16-byte pieces of a weight row of the last layer
    const int orow = tid / CP, oc8 = tid % CP;
    const int srow = wave * 32 + (lane >> 3), sc8 = (lane & 7) * 8;     // rows srow + 8 i of the shortcut and of the result
    uint4 w3r[NB], wpr[PROJ ? 2 : 1], w1r[CHAIN ? NB : 1], rres[PROJ ? 1 : 4];
    auto fetch_pass = [&](int n0) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const int n = n0 + orow + (NT / CP) * i;
            w3r[i] = load16(rs_w3, n < out && oc8 * 8 < mid ? (uint32_t)(n * a.mid_full + oc8 * 8) * 2 : OOB);
        }
        if constexpr (PROJ) {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int n = n0 + (tid >> 3) + 32 * i, k = (tid & 7) * 8;
                wpr[i] = load16(rs_wp, n < out && k < kx ? (uint32_t)(n * a.x_full + k) * 2 : OOB);
            }
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int z = rowZ[srow + 8 * i];
                rres[i] = make_uint4(0, 0, 0, 0);
                if (z >= 0 && n0 + sc8 < out) rres[i] = *(const uint4*)(a.shortcut + z + n0 + sc8);
            }
        }
        if constexpr (CHAIN) {
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                const int n = (tid >> 3) + 32 * i, k = n0 + (tid & 7) * 8;
                w1r[i] = load16(rs_w1, n < next && k < out ? (uint32_t)(n * a.out_full + k) * 2 : OOB);
            }
        }
    };

    bf16x8_t xf[PROJ ? 4 : 1];                         // PROJ: the stage's input at this lane's pixel, as operands
    auto fetch_x = [&]() {
        if constexpr (PROJ) {
            const __amdgpu_buffer_rsrc_t rs_x = __builtin_amdgcn_make_buffer_rsrc((void*)a.x, 0, 0x7fffffff, 0x00020000);
#pragma unroll
            for (int k = 0; k < 4; ++k) xf[k] = __builtin_bit_cast(bf16x8_t, load16(rs_x, k * 16 + lhi * 8 < kx ? xoff : OOB, k * 32));
        }
    };

    const int nph = (mid + 31) / 32 * 3;
    store_phase(0);
    __syncthreads();
    auto products = [&](int c, int u) __attribute__((always_inline)) {
        const int ksteps = mid - c * 32 > 16 ? 2 : 1;
        if constexpr (NB == 2) {
            if (mid > 32) taps(std::integral_constant<int, 2>(), u, ksteps);
            else taps(std::integral_constant<int, 1>(), u, ksteps);
        } else {
            if (mid > 64) taps(std::integral_constant<int, NB>(), u, ksteps);
            else taps(std::integral_constant<int, 2>(), u, ksteps);
        }
    };
    int c = 0, u = 0;
    for (int ph = 1; ph < nph; ++ph) {
        const int un = u == 2 ? 0 : u + 1, cn = u == 2 ? c + 1 : c;
        load_phase(cn, un);
        products(c, u);
        __syncthreads();
        store_phase(un);
        __syncthreads();
        c = cn;
        u = un;
    }
    fetch_pass(0);                                     // in flight during the last phase
    products(c, 2);
    __syncthreads();
    fetch_x();
    // y2 of this lane's pixel as operands: [k-step], channels 16 k + 8 lhi ..
    bf16x8_t y2[2 * NB];
#pragma unroll
    for (int t = 0; t < NB; ++t)
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            uint2 q2[2];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int q = 2 * h + j, ch = t * 32 + q * 8 + lhi * 4;
                q2[j] = make_uint2(0, 0);              // (behind the slice zeros, whatever the stored tables and filters hold)
                if (t * 32 + q * 8 < mid) {
                    const float4 s4 = *(const float4*)(cst2 + ch), h4 = *(const float4*)(cst2 + 32 * NB + ch);
                    q2[j].x = f2bf2(fmaxf(acc[t][4 * q] * s4.x + h4.x, 0.f), fmaxf(acc[t][4 * q + 1] * s4.y + h4.y, 0.f));
                    q2[j].y = f2bf2(fmaxf(acc[t][4 * q + 2] * s4.z + h4.z, 0.f), fmaxf(acc[t][4 * q + 3] * s4.w + h4.w, 0.f));
                }
            }
            const auto a0 = __builtin_amdgcn_permlane32_swap(q2[0].x, q2[1].x, false, false);
            const auto a1 = __builtin_amdgcn_permlane32_swap(q2[0].y, q2[1].y, false, false);
            y2[2 * t + h] = __builtin_bit_cast(bf16x8_t, make_uint4(a0[0], a1[0], a0[1], a1[1]));
        }

    // ---- passes of 64 output columns ------------------------------------------------------------------------------------------
    f32x16_t acc1[CHAIN ? NB : 1];
#pragma unroll
    for (int t = 0; t < (CHAIN ? NB : 1); ++t)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc1[t][v] = 0.f;
    char *W3 = smem + TILE_BYTES, *WP = W3 + L::W3, *W1 = WP + L::WP;
    float* colsum = (float*)(smem + L::SUMS);
    char* my_row = tile + prow * 128;
    const int px7 = prow & 7;
    for (int n0 = 0; n0 < out; n0 += 64) {
        if (n0) __syncthreads();      // the last pass's weights have been read
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const int n = orow + (NT / CP) * i;
            *(uint4*)(W3 + ((oc8 >> 2) * 64 + n) * 64 + (((oc8 & 3) ^ sw(n)) * 16)) = w3r[i];
        }
        if constexpr (PROJ) {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int n = (tid >> 3) + 32 * i, c = tid & 7;
                *(uint4*)(WP + ((c >> 2) * 64 + n) * 64 + (((c & 3) ^ sw(n)) * 16)) = wpr[i];
            }
        } else {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int r = srow + 8 * i;
                *(uint4*)(tile + r * 128 + (((lane & 7) ^ (r & 7)) * 16)) = rres[i];
            }
        }
        if constexpr (CHAIN) {
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                const int n = (tid >> 3) + 32 * i, c = tid & 7;
                *(uint4*)(W1 + ((c >> 2) * 32 * NB + n) * 64 + (((c & 3) ^ sw(n)) * 16)) = w1r[i];
            }
        }
        __syncthreads();
        if (n0 + 64 < out) fetch_pass(n0 + 64);        // in flight during this pass
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            f32x16_t o, op;
            auto product = [&](f32x16_t& o, const char* w, const bf16x8_t f, int k) __attribute__((always_inline)) {
                const bf16x8_t wf = *(const bf16x8_t*)(w + ((k >> 1) * 64 + t * 32 + l32) * 64 + ((((k & 1) * 2 + lhi) ^ sw(l32)) * 16));
                o = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf, f, o, 0, 0, 0);
            };
            uint2 sc[4];                               // the projection's rounded results
            if constexpr (PROJ) {
#pragma unroll
                for (int v = 0; v < 16; ++v) op[v] = 0.f;
#pragma unroll
                for (int k = 0; k < 4; ++k) product(op, WP, xf[k], k);      // (zeros behind the slice on both sides)
            }
#pragma unroll
            for (int v = 0; v < 16; ++v) o[v] = 0.f;
#pragma unroll
            for (int k = 0; k < 2 * NB; k += 2)
                if (k * 16 < mid) {
                    product(o, W3, y2[k], k);
                    product(o, W3, y2[k + 1], k + 1);
                }
            if constexpr (PROJ) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int col = n0 + t * 32 + q * 8 + lhi * 4;
                    const float4 s4 = *(const float4*)(cst + 2 * L::N_OUT + col), h4 = *(const float4*)(cst + 3 * L::N_OUT + col);
                    sc[q].x = f2bf2(op[4 * q] * s4.x + h4.x, op[4 * q + 1] * s4.y + h4.y);
                    sc[q].y = f2bf2(op[4 * q + 2] * s4.z + h4.z, op[4 * q + 3] * s4.w + h4.w);
                }
            }
            // batch-norm, shortcut, ReLU in place on this lane's runs of four channels
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int col = n0 + t * 32 + q * 8 + lhi * 4;
                const float4 s4 = *(const float4*)(cst + col), h4 = *(const float4*)(cst + L::N_OUT + col);
                float v[4] = {o[4 * q] * s4.x + h4.x, o[4 * q + 1] * s4.y + h4.y, o[4 * q + 2] * s4.z + h4.z, o[4 * q + 3] * s4.w + h4.w};
                uint2* tp = (uint2*)(my_row + (((t * 4 + q) ^ px7) * 16) + lhi * 8);
                add_bf16x4(v, PROJ ? sc[q] : *tp);
                *tp = make_uint2(f2bf2(fmaxf(v[0], 0.f), fmaxf(v[1], 0.f)), f2bf2(fmaxf(v[2], 0.f), fmaxf(v[3], 0.f)));
            }
        }
        wave_sync();
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int r = srow + 8 * i, z = rowZ[r];
            if (z >= 0 && n0 + sc8 < out) *(uint4*)(a.z + z + n0 + sc8) = *(const uint4*)(tile + r * 128 + (((lane & 7) ^ (r & 7)) * 16));
        }
        if constexpr (!CHAIN) {
            if (a.sums) {
                // sums over this wavefront's rows (as stored), 8 columns a lane, then over the 8 lanes that share the columns
                float t[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int r = srow + 8 * i;
                    if (rowZ[r] < 0) continue;
                    const uint4 q = *(const uint4*)(tile + r * 128 + (((lane & 7) ^ (r & 7)) * 16));
                    const uint32_t u[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        t[2 * k] += __uint_as_float(u[k] << 16);
                        t[2 * k + 1] += __uint_as_float(u[k] & 0xffff0000u);
                    }
                }
#pragma unroll
                for (int k = 0; k < 8; ++k) t[k] = sum_of_8(t[k]);
                if (lane < 8) {
                    float* p = colsum + wave * L::N_OUT + n0 + lane * 8;
                    *(float4*)p = make_float4(t[0], t[1], t[2], t[3]);
                    *(float4*)(p + 4) = make_float4(t[4], t[5], t[6], t[7]);
                }
            }
        }
        if constexpr (CHAIN) {
            if (next > 0) {
                const int nk = out - n0;
#pragma unroll 1
                for (int k0 = 0; k0 < 4 && k0 * 16 < nk; k0 += 2)
#pragma unroll
                    for (int k = k0; k < k0 + 2; ++k) {
                        bf16x8_t pf = *(const bf16x8_t*)(my_row + (((2 * k + lhi) ^ px7) * 16));
                        // (columns behind the slice are not finite for certain)
                        if (k * 16 + lhi * 8 >= nk) pf = __builtin_bit_cast(bf16x8_t, make_uint4(0, 0, 0, 0));
#pragma unroll
                        for (int t = 0; t < NB; ++t) {
                            const bf16x8_t wf = *(const bf16x8_t*)(W1 + ((k >> 1) * 32 * NB + t * 32 + l32) * 64 + ((((k & 1) * 2 + lhi) ^ sw(l32)) * 16));
                            acc1[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf, pf, acc1[t], 0, 0, 0);
                        }
                    }
            }
        }
        wave_sync();
    }
    if constexpr (!CHAIN) {
        if (!a.sums) return;
        __syncthreads();
        // a tile starts at a multiple of 64 rows of a sample, so either half is one piece of one sample, whoever its neighbours are
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int m = grow0 + h * SUM_ROWS, sl = m / rows;
            if (m >= rows_g) break;
            float* to = a.sums + ((int64_t)(slot0 + sl) * (rows / SUM_ROWS) + (m - sl * rows) / SUM_ROWS) * a.out_full;
            for (int i = tid; i < out; i += NT) to[i] = colsum[2 * h * L::N_OUT + i] + colsum[(2 * h + 1) * L::N_OUT + i];
        }
        return;
    }
    if constexpr (CHAIN) {
        if (next <= 0) return;
        // the next block's input leaves through the same rows, 64 columns at a time
#pragma unroll
        for (int hb = 0; hb < NB / 2; ++hb) {
            if (hb * 64 >= next) continue;
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int ch = hb * 64 + t * 32 + q * 8 + lhi * 4;
                    const float4 s4 = *(const float4*)(cst2 + 64 * NB + ch), h4 = *(const float4*)(cst2 + 96 * NB + ch);
                    const f32x16_t& v = acc1[2 * hb + t];
                    *(uint2*)(my_row + (((t * 4 + q) ^ px7) * 16) + lhi * 8) =
                        make_uint2(f2bf2(fmaxf(v[4 * q] * s4.x + h4.x, 0.f), fmaxf(v[4 * q + 1] * s4.y + h4.y, 0.f)),
                                   f2bf2(fmaxf(v[4 * q + 2] * s4.z + h4.z, 0.f), fmaxf(v[4 * q + 3] * s4.w + h4.w, 0.f)));
                }
            wave_sync();
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int r = srow + 8 * i, y = row1[r];
                if (y >= 0 && hb * 64 + sc8 < next)
                    *(uint4*)(a.y1_next + y + hb * 64 + sc8) = *(const uint4*)(tile + r * 128 + (((lane & 7) ^ (r & 7)) * 16));
            }
            wave_sync();
        }
    }
}

template <int NB, bool PROJ, bool CHAIN>
int32_t launch(const BneckArgs& a, int32_t max_mtiles, hipStream_t s) {
    using L = Layout<NB, PROJ, CHAIN>;
    constexpr int MOST = CHAIN ? L::SMEM : L::SMEM_SUMS;
    const int SMEM = !CHAIN && a.sums ? L::SMEM_SUMS : L::SMEM;
    const int32_t rc = ds_reserve_lds((const void*)bneck_kernel<NB, PROJ, CHAIN>, MOST, "bottleneck block");
    if (rc) return rc;
    ProfScope prof(DS_K_CONV3, s);
    hipLaunchKernelGGL((bneck_kernel<NB, PROJ, CHAIN>), dim3((unsigned)((max_mtiles + 63) / 64 * 64)), dim3(NT), SMEM, s, a, max_mtiles);
    DS_CHECK_LAUNCH("bottleneck block");
    return DS_OK;
}

int blocks_of(const BneckArgs& a) {
    for (int t = 0; t < a.gt.T; ++t)
        if (a.gt.k_in[t] > 64 || (a.w1 && a.next[t] > 64)) return 4;
    return 2;
}

}  // namespace

bool ds_bneck_runs(const BneckArgs& a, int32_t B, int32_t max_mtiles) {
    if (BM + 2 * (a.W + 1) > RMAX || (a.sums && (a.w1 || (a.H * a.W) % SUM_ROWS))) return false;
    int mmax = 0, omax = 0, xmax = 0, nmax = 0;
    for (int t = 0; t < a.gt.T; ++t) {
        const int x = a.x ? a.kx[t] : 0, n = a.w1 ? a.next[t] : 0;
        if ((a.gt.k_in[t] | a.gt.k_out[t] | x | n) % 8) return false;
        mmax = a.gt.k_in[t] > mmax ? a.gt.k_in[t] : mmax;
        omax = a.gt.k_out[t] > omax ? a.gt.k_out[t] : omax;
        xmax = x > xmax ? x : xmax;
        nmax = n > nmax ? n : nmax;
    }
    const int nb = blocks_of(a);
    if (mmax > 128 || nmax > 128 || omax > 128 * nb || xmax > 64 || (a.x && nb != 2)) return false;
    if ((a.mid_full | a.out_full | (a.x ? a.x_full : 0)) % 8) return false;     // 16-byte pieces of the stored filters
    // 16-byte pieces everywhere; 32-bit offsets
    if (((a.y1_ss | a.z_ss | (a.x ? a.x_ss : 0)) % 8) ||
        (((uintptr_t)a.y1 | (uintptr_t)a.w2 | (uintptr_t)a.w3 | (uintptr_t)a.w1 | (uintptr_t)a.wp | (uintptr_t)a.x | (uintptr_t)a.z |
          (uintptr_t)a.shortcut | (uintptr_t)a.y1_next | (uintptr_t)a.s1 | (uintptr_t)a.h1) & 15))
        return false;
    const int64_t lim = 0x7fffffffLL;
    if (B * a.y1_ss * 2 >= lim || B * a.z_ss >= lim || (a.x && B * a.x_ss * 2 >= lim) || 9LL * a.mid_full * (mmax + 1) * 2 >= lim ||
        (int64_t)a.out_full * (nmax + 1) * 2 >= lim || ((int64_t)(a.x ? a.x_full : 0) + a.mid_full) * (omax + 1) * 2 >= lim)
        return false;
    // A workgroup is a chain of 3 phases a 32-channel chunk and a pass per 64 output columns, against three launches whose tiles spread
    // over more workgroups.  DS-ResNet, us a pass, separate launches / here: slices up to 64 channels 1 image (25 tiles) 366 / 371, 2 images
    // (50) 439 / 433, 3 images (75) 527 / 509, 16 images 716 / 682; up to 128 channels 24 images (162 tiles) 767 / 800, 33 images (217)
    // 863 / 882, 40 images (260) 927 / 932, 48 images (309) 1005 / 1004, 64 images (407) 1181 / 1142, 96 images 1432 / 1389.  Parts of a
    // batch that run side by side count together: 160 images in four parts (260 tiles each) 1987 / 1924.
    return (int64_t)max_mtiles * (a.crowd > 1 ? a.crowd : 1) >= (nb == 2 ? 40 : 300);
}

int32_t ds_launch_bneck(const BneckArgs& a, int32_t B, int32_t max_mtiles, hipStream_t s) {
    if (!ds_bneck_runs(a, B, max_mtiles)) return DS_EUNSUPPORTED;
    if (blocks_of(a) == 4) return a.w1 ? launch<4, false, true>(a, max_mtiles, s) : launch<4, false, false>(a, max_mtiles, s);
    if (a.x) return a.w1 ? launch<2, true, true>(a, max_mtiles, s) : launch<2, true, false>(a, max_mtiles, s);
    return a.w1 ? launch<2, false, true>(a, max_mtiles, s) : launch<2, false, false>(a, max_mtiles, s);
}
