// Grouped prefix-slice 3x3 convolution (stride 1, padding 1) as an implicit GEMM whose input patch
// is staged once per channel chunk (filter slicing, Section 3.3 Eq. 9; split batch-norm, Eq. 14).
//
// gemm_kernel walks the 9 taps as 9 separate reduction slabs and fetches the 128 shifted input
// pixels of each tap from L2 again.  Here a workgroup (same 128-pixel x 64-filter tile, same
// epilogue) loads, for every 32-channel chunk, the contiguous run of input pixels that its 128
// output pixels touch -- pixel indices m - (W+1) .. m + 127 + (W+1) in the group's row-major pixel
// order, 128 + 2 (W+1) rows -- once into LDS, and every tap reads its operand rows from that patch
// at a fixed row offset ((u-1) W + (v-1)); lanes whose tap falls outside the image (or the group)
// read a row of zeros instead.  A tap that is inside the image never leaves the sample, so the
// linear pixel order needs no per-sample bookkeeping.  The weights of one filter row (3 taps) are
// staged per phase: 12 matrix instructions per wavefront between barriers instead of 4, and the
// activation traffic from L2 drops from 9 x 128 rows per chunk to 128 + 2 (W+1).
// Launches of fewer workgroups than run at once deal the chunks of a tile to two or four shares of four wavefronts, each with slabs of
// its own in LDS; the partial tiles are added there in share order.
#include "gelu.h"

namespace {

constexpr int BM = DS_GEMM_BM, BN = 64, NT = 256;   // NT: threads of a share of the reduction
constexpr int RMAX = 248;                      // patch rows: 128 + 2 (W + 1), so W <= 59
constexpr int ZROW = RMAX;                     // one more row, all zeros
constexpr int TPP = 3;                         // taps staged per phase: 3 (one filter row) or 9 (the whole filter)
constexpr int PPC = 9 / TPP;                   // phases per channel chunk
constexpr int A_BYTES = (RMAX + 1) * 64, B_BYTES = TPP * BN * 64;
constexpr int SROWS = 16, ST_LD = BN + 4, STAGE_BYTES = 4 * SROWS * ST_LD * 4;
constexpr int TABLE_BYTES = BM * 16;
// LDS of a share: its slabs, and with several shares its partial tile
constexpr int main_bytes(int ks) {
    const int m = A_BYTES + B_BYTES > STAGE_BYTES ? A_BYTES + B_BYTES : STAGE_BYTES;
    return ks > 1 && BM * ST_LD * 4 > m ? BM * ST_LD * 4 : m;
}
constexpr int smem_bytes(int ks) { return ks * main_bytes(ks) + TABLE_BYTES; }
constexpr int NR = (RMAX * 4 + NT - 1) / NT;   // 16-byte patch loads per thread and chunk

// chunk c of a 64-byte LDS row r is stored at position c ^ sw(r): any run of consecutive rows read
// with one chunk column spreads over the banks, whatever row the run starts at, for access groups of
// 8 lanes (128 bytes) and of 16 lanes (256 bytes) alike -- a key of (r >> 1) & 3 serves only the former
// and cost 40 % of the LDS cycles in conflicts
__device__ __forceinline__ int sw(int r) { return ((r >> 1) ^ (r >> 2)) & 3; }

// KS: shares of the reduction, four wavefronts each; a share takes every KS-th chunk of 32 channels
template <bool HASR, int KS>
__global__ __launch_bounds__(NT * KS) void conv3_kernel(const GemmArgs a, const int ny, const int max_mtiles) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int share = KS > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x / NT) : 0;
    char* As = smem + share * main_bytes(KS);          // [RMAX + 1][32] bf16
    char* Bs = As + A_BYTES;                           // [TPP][BN][32] bf16
    long long* rowC = (long long*)(smem + KS * main_bytes(KS));
    long long* rowR = rowC + BM;
    constexpr uint32_t OOB = 0x80000000u;

    const int j = (int)(blockIdx.x >> 3);
    const int jm = j / ny, y = j - jm * ny;
    const int mt = jm * 8 + (int)(blockIdx.x & 7);
    if (mt >= max_mtiles) return;
    const GroupLanes lanes(a.gt);
    const bf16_t *A = a.A, *Wt = a.Wt, *res = a.R;
    void* C = a.C;
    const float *scale = a.scale, *shift = a.shift;
    const int32_t *a_index = a.a_index, *c_index = a.c_index;
    int64_t a_ss = a.a_sample_stride, c_ss = a.c_sample_stride, r_ss = a.r_sample_stride;
    int a_ld = a.a_ld, c_ld = a.c_ld, r_ld = a.r_ld, c_row0 = a.c_row0, r_use = a.r_use_index, w_ld = (int)a.w_ld;
    int w_tap = (int)a.w_tap_stride, tab_ld = a.tab_ld, W = a.W, H = a.H, rows = a.rows, act = a.act, out_f32 = a.out_f32;
    const int4 me = ds_tile_record(a, mt);
    ds_hold(A, Wt, res, C, scale, shift, a_index, c_index, a_ss, c_ss, r_ss, a_ld, c_ld, r_ld, c_row0, r_use, w_ld, w_tap, tab_ld, W, H,
            rows, act, out_f32);
    if (me.x < 0) return;
    const __amdgpu_buffer_rsrc_t rsrc_a = __builtin_amdgcn_make_buffer_rsrc((void*)A, 0, 0x7fffffff, 0x00020000);
    const __amdgpu_buffer_rsrc_t rsrc_w = __builtin_amdgcn_make_buffer_rsrc((void*)Wt, 0, 0x7fffffff, 0x00020000);
    const int g = me.x, grow0 = me.y, slot0 = me.z, rows_g = me.w;
    const int k_in = lanes.k_in(g), k_out = lanes.k_out(g);
    if (k_in <= 0 || k_out <= 0) return;
    const int n0 = y * BN;
    if (n0 >= k_out) return;

    const int tid = threadIdx.x & (NT - 1);            // of the share
    if (a_ld <= 0) a_ld = k_in;
    if (c_ld <= 0) c_ld = k_out;
    if (r_ld <= 0) r_ld = k_out;
    const int halo = W + 1, R = BM + 2 * halo;

    if (tid < 4) *(uint4*)(As + ZROW * 64 + tid * 16) = make_uint4(0, 0, 0, 0);

    // ---- patch loader: item e = tid + 256 i is chunk (e & 3) of patch row (e >> 2) --------------
    const int lchunk = tid & 3;
    uint32_t poff[NR];
#pragma unroll
    for (int i = 0; i < NR; ++i) {
        const int jr = (tid + NT * i) >> 2;
        const int L = grow0 - halo + jr;              // pixel index in the group's row-major order
        uint32_t o = OOB;
        if (jr < R && L >= 0 && L < rows_g) {
            const int sl = L / rows;
            const int p = L - sl * rows;
            const int slot = slot0 + sl;
            const int sa = a_index ? a_index[slot] : slot;
            o = (uint32_t)(((long long)sa * a_ss + (long long)p * a_ld + lchunk * 8) * 2);
        }
        poff[i] = o;
    }
    // ---- weight loader: chunk (tid & 3) of filter row n0 + (tid >> 2), one load per tap ---------
    const int wn_row = tid >> 2;
    const uint32_t woff = (n0 + wn_row) < k_out ? (uint32_t)((n0 + wn_row) * w_ld + lchunk * 8) * 2 : OOB;

    uint4 ra[NR], rb[TPP];
    auto load_phase = [&](int c, int u) {
        const int kc = c * 32;
        const bool kok = kc + lchunk * 8 < k_in;
        if (u == 0) {
#pragma unroll
            for (int i = 0; i < NR; ++i) {
                const auto t = __builtin_amdgcn_raw_buffer_load_b128(rsrc_a, (int)(kok ? poff[i] : OOB), kc * 2, 0);
                ra[i] = make_uint4(t[0], t[1], t[2], t[3]);
            }
        }
#pragma unroll
        for (int v = 0; v < TPP; ++v) {
            const int soff = ((u * TPP + v) * w_tap + kc) * 2;
            const auto t = __builtin_amdgcn_raw_buffer_load_b128(rsrc_w, (int)(kok ? woff : OOB), soff, 0);
            rb[v] = make_uint4(t[0], t[1], t[2], t[3]);
        }
    };
    auto store_phase = [&](int u) {
        if (u == 0) {
#pragma unroll
            for (int i = 0; i < NR; ++i) {
                const int jr = (tid + NT * i) >> 2;
                if (jr < R) *(uint4*)(As + jr * 64 + ((lchunk ^ sw(jr)) * 16)) = ra[i];
            }
        }
#pragma unroll
        for (int v = 0; v < TPP; ++v) *(uint4*)(Bs + (v * BN + wn_row) * 64 + ((lchunk ^ sw(wn_row)) * 16)) = rb[v];
    };

    // the first patch and filter-row loads are requested as soon as their addresses are known: everything below (output
    // row table, tap mask, epilogue constants) is worked out while they travel
    load_phase(share, 0);

    if (threadIdx.x < BM) {
        const int m = grow0 + tid;
        long long rc = -1, rr = 0;
        if (m < rows_g) {
            const int sl = m / rows;
            const int p = m - sl * rows;
            const int slot = slot0 + sl;
            const int cs = c_index ? c_index[slot] : slot;
            rc = (long long)cs * c_ss + (long long)(p + c_row0) * c_ld;
            rr = (long long)(r_use ? cs : 0) * r_ss + (long long)(p + c_row0) * r_ld;
        }
        rowC[tid] = rc;
        rowR[tid] = rr;
    }
    const int wave = tid >> 6, lane = tid & 63, l32 = lane & 31, lhi = lane >> 5;
    // ---- this lane's output pixel: which taps are inside the image ---------------------------
    const int trow = wave * 32 + l32;
    int tapmask = 0;
    {
        const int m = grow0 + trow;
        if (m < rows_g) {
            const int p = m % rows;
            const int oy = p / W, ox = p - oy * W;
#pragma unroll
            for (int u = 0; u < 3; ++u)
#pragma unroll
                for (int v = 0; v < 3; ++v) {
                    const int iy = oy + u - 1, ix = ox + v - 1;
                    if (iy >= 0 && iy < H && ix >= 0 && ix < W) tapmask |= 1 << (u * 3 + v);
                }
        }
    }

    f32x16_t acc[2];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[t][v] = 0.f;

    // epilogue constants and residual rows, fetched early so that their latency hides behind the loop
    constexpr int COLS = BN, CG = COLS / 4, RPP = 64 / CG, PASSES = 32 / SROWS, VPP = 16 / PASSES;
    const int cg = lane % CG, rr0 = lane / CG;
    const int ncol = n0 + cg * 4;
    const bool nok = ncol < k_out;
    float sc[4] = {1.f, 1.f, 1.f, 1.f}, sh[4] = {0.f, 0.f, 0.f, 0.f};
    if (nok) {
        const long long ti = (long long)lanes.row(g) * tab_ld + ncol;
        if (scale) {
            const float4 t = *(const float4*)(scale + ti);
            sc[0] = t.x; sc[1] = t.y; sc[2] = t.z; sc[3] = t.w;
        }
        if (shift) {
            const float4 t = *(const float4*)(shift + ti);
            sh[0] = t.x; sh[1] = t.y; sh[2] = t.z; sh[3] = t.w;
        }
    }
    __syncthreads();                                   // row table visible
    // rows that this thread finishes: one share 8 of its wavefront's own, several shares every 16 KS-th of the tile
    constexpr int NE = KS == 1 ? PASSES * (SROWS / RPP) : BM / (16 * KS);
    auto my_row = [&](int i) {
        if constexpr (KS == 1) return wave * 32 + (i / (SROWS / RPP)) * SROWS + rr0 + (i % (SROWS / RPP)) * RPP;
        else return ((int)threadIdx.x >> 4) + i * 16 * KS;
    };
    uint2 rres[HASR ? NE : 1];
    if constexpr (HASR) {
#pragma unroll
        for (int i = 0; i < NE; ++i) {
            const int r = my_row(i);
            rres[i] = make_uint2(0, 0);
            if (nok && rowC[r] >= 0) rres[i] = *(const uint2*)(res + rowR[r] + ncol);
        }
    }
    // four channels of a row: batch-norm, residual, activation, store
    auto finish = [&](const float4 t, long long coff, const uint2 q) {
        float val[4] = {t.x * sc[0] + sh[0], t.y * sc[1] + sh[1], t.z * sc[2] + sh[2], t.w * sc[3] + sh[3]};
        if constexpr (HASR) {
            val[0] += __uint_as_float(q.x << 16);
            val[1] += __uint_as_float(q.x & 0xffff0000u);
            val[2] += __uint_as_float(q.y << 16);
            val[3] += __uint_as_float(q.y & 0xffff0000u);
        }
        if (act == DS_ACT_RELU) {
#pragma unroll
            for (int e = 0; e < 4; ++e) val[e] = fmaxf(val[e], 0.f);
        } else if (act == DS_ACT_GELU) {
#pragma unroll
            for (int e = 0; e < 4; ++e) val[e] = gelu_erf(val[e]);
        }
        if (out_f32) *(float4*)((float*)C + coff + ncol) = make_float4(val[0], val[1], val[2], val[3]);
        else *(uint2*)((bf16_t*)C + coff + ncol) = make_uint2(f2bf2(val[0], val[1]), f2bf2(val[2], val[3]));
    };

    // every share goes through as many phases; one past its last chunk multiplies zeros
    const int nph = (((k_in + 31) / 32 + KS - 1) / KS) * PPC;
    store_phase(0);
    __syncthreads();
    int c = share, u = 0;
    for (int ph = 0; ph < nph; ++ph) {
        int cn = c, un = u + 1;
        if (un == PPC) {
            un = 0;
            cn += KS;
        }
        const bool more = ph + 1 < nph;
        if (more) load_phase(cn, un);
#pragma unroll
        for (int v = 0; v < TPP; ++v) {
            const int tap = u * TPP + v;
            const int tu = tap / 3, tv = tap - tu * 3;
            const int arow = ((tapmask >> tap) & 1) ? trow + halo + (tu - 1) * W + (tv - 1) : ZROW;
            const char* ap = As + arow * 64;
            const int fa = sw(arow);
#pragma unroll
            for (int kk = 0; kk < 2; ++kk) {
                const int ch = kk * 2 + lhi;
                const bf16x8_t af = *(const bf16x8_t*)(ap + ((ch ^ fa) * 16));
                bf16x8_t bfr[2];
#pragma unroll
                for (int t = 0; t < 2; ++t) {
                    const int nr = t * 32 + l32;
                    bfr[t] = *(const bf16x8_t*)(Bs + (v * BN + nr) * 64 + ((ch ^ sw(nr)) * 16));
                }
#pragma unroll
                for (int t = 0; t < 2; ++t) acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af, bfr[t], acc[t], 0, 0, 0);
            }
        }
        __syncthreads();
        if (more) {
            store_phase(un);
            __syncthreads();
        }
        c = cn;
        u = un;
    }

    if constexpr (KS > 1) {
        // ---- partial tiles to LDS, added in share order ------------------------------------------------------------------
        // (the loop's last barrier has retired every read of the slabs they take the place of)
        float* part = (float*)As;
#pragma unroll
        for (int tn = 0; tn < 2; ++tn)
#pragma unroll
            for (int v = 0; v < 16; ++v) part[(wave * 32 + 8 * (v >> 2) + 4 * lhi + (v & 3)) * ST_LD + tn * 32 + l32] = acc[tn][v];
        __syncthreads();
#pragma unroll
        for (int i = 0; i < NE; ++i) {
            const int r = my_row(i);
            const long long coff = rowC[r];
            if (!nok || coff < 0) continue;
            float4 t = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
            for (int k = 0; k < KS; ++k) {
                const float4 q = *(const float4*)((const float*)(smem + k * main_bytes(KS)) + r * ST_LD + cg * 4);
                t.x += q.x; t.y += q.y; t.z += q.z; t.w += q.w;
            }
            finish(t, coff, rres[HASR ? i : 0]);
        }
    } else {
        // ---- epilogue through LDS: each lane finishes 4 consecutive channels of one row -----------
        // staging rows are private to a wavefront and the loop's last barrier has retired every read of the tiles they
        // alias: between the passes only the compiler has to be kept from moving LDS accesses
        auto wave_sync = [] {
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
            __builtin_amdgcn_wave_barrier();
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
        };
        float* st = (float*)smem + wave * SROWS * ST_LD;
#pragma unroll
        for (int ps = 0; ps < PASSES; ++ps) {
#pragma unroll
            for (int tn = 0; tn < 2; ++tn)
#pragma unroll
                for (int vv = 0; vv < VPP; ++vv) {
                    const int v = ps * VPP + vv;
                    const int lr = 8 * ((v >> 2) - ps * (4 / PASSES)) + 4 * lhi + (v & 3);
                    st[lr * ST_LD + tn * 32 + l32] = acc[tn][v];
                }
            wave_sync();
            if (nok) {
#pragma unroll
                for (int rr = rr0; rr < SROWS; rr += RPP) {
                    const long long coff = rowC[wave * 32 + ps * SROWS + rr];
                    if (coff < 0) continue;
                    finish(*(const float4*)(st + rr * ST_LD + cg * 4), coff, rres[HASR ? ps * (SROWS / RPP) + (rr - rr0) / RPP : 0]);
                }
            }
            wave_sync();
        }
    }
}

template <bool HASR, int KS>
int32_t launch(const GemmArgs& a, int32_t max_mtiles, int32_t max_kout, hipStream_t s) {
    auto kern = conv3_kernel<HASR, KS>;
    {
        const int32_t rc = ds_reserve_lds((const void*)kern, smem_bytes(KS), "sliced 3x3 conv");
        if (rc) return rc;
    }
    const int ny = (max_kout + BN - 1) / BN;
    const unsigned grid = (unsigned)(((max_mtiles + 7) / 8) * ny * 8);
    ProfScope prof(DS_K_CONV3, s);
    hipLaunchKernelGGL(kern, dim3(grid), dim3(NT * KS), smem_bytes(KS), s, a, ny, max_mtiles);
    DS_CHECK_LAUNCH("sliced 3x3 conv");
    return DS_OK;
}

}  // namespace

// 3x3, stride 1, padding 1, one segment, maps up to 59 pixels wide; DS_EUNSUPPORTED otherwise
int32_t ds_launch_conv3(const GemmArgs& a, int32_t max_mtiles, int32_t max_kout, hipStream_t s) {
    if (a.K != 3 || a.stride != 1 || a.pad != 1 || a.n_seg != 1 || a.Ho != a.H || a.Wo != a.W || a.rows != a.H * a.W ||
        BM + 2 * (a.W + 1) > RMAX)
        return DS_EUNSUPPORTED;
    if (((long long)max_kout * a.w_ld + 9 * a.w_tap_stride) * 2 >= 0x7fffffffLL) return DS_EUNSUPPORTED;   // 32-bit weight offsets
    int kmax = 0;
    for (int t = 0; t < a.gt.T; ++t) kmax = a.gt.k_in[t] > kmax ? a.gt.k_in[t] : kmax;
    const int64_t wgs = (int64_t)max_mtiles * ((max_kout + BN - 1) / BN) * (a.crowd > 1 ? a.crowd : 1);
    // Shares of the reduction.  A workgroup is a chain of 3 phases a chunk, about 0.9 us each, whatever else runs; with fewer
    // workgroups than the compute units could hold, shares shorten it.  DS-ResNet, 33 images, us a launch, one share -> here: 28x28
    // maps (up to 4 chunks, 436 workgroups) 14.8 -> 12.3, 14x14 (8, 268) 22.2 -> 17.1, 7x7 (16, 232) 37.3 -> 24.0; 64 images 14x14
    // 24.4 -> 18.3, 7x7 40.8 -> 28.  Twice these lines: 33 / 64 / 96 images 905 / 1248 / 1523 -> 931 / 1291 / 1515 us a pass (the shares of a
    // workgroup wait for each other); four shares of 16 chunks up to 512 workgroups in place of 256: 64 / 96 images 1253 / 1530 -> 1248 / 1523.  Parts of a batch that run side by side count together: 256 images in
    // four parts 2894 us, 3097 with shares.
    const int ks = kmax > 64 && wgs <= (kmax > 256 ? 512 : 256) ? 4 : kmax > 32 && wgs <= 512 ? 2 : 1;
#define DS_CONV3(KS) (a.R ? launch<true, KS>(a, max_mtiles, max_kout, s) : launch<false, KS>(a, max_mtiles, max_kout, s))
    return ks == 4 ? DS_CONV3(4) : ks == 2 ? DS_CONV3(2) : DS_CONV3(1);
#undef DS_CONV3
}
