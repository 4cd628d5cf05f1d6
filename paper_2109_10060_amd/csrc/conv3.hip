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
#include "tile_out.h"

namespace {

constexpr int BM = DS_GEMM_BM, BN = 64, NT = 256;   // NT: threads of a share of the reduction
constexpr int RMAX = 248;                      // patch rows: 128 + 2 (W + 1), so W <= 59
constexpr int ZROW = RMAX;                     // one more row, all zeros
constexpr int TPP = 3;                         // taps staged per phase: 3 (one filter row) or 9 (the whole filter)
constexpr int PPC = 9 / TPP;                   // phases per channel chunk
constexpr int A_BYTES = (RMAX + 1) * 64, B_BYTES = TPP * BN * 64;
constexpr int ST_LD = BN + 8, STAGE_BYTES = 4 * 32 * ST_LD * 2;   // bf16 stage: an odd number of 16-byte chunks a row
constexpr int PT_LD = BN + 4;                  // of a share's partial tile (fp32)
constexpr int TABLE_BYTES = BM * 16 + 2 * BN * 4;   // output and residual rows, scale and shift
// LDS of a share: its slabs, and with several shares its partial tile
constexpr int main_bytes(int ks) {
    const int m = A_BYTES + B_BYTES > STAGE_BYTES ? A_BYTES + B_BYTES : STAGE_BYTES;
    return ks > 1 && BM * PT_LD * 4 > m ? BM * PT_LD * 4 : m;
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
__global__ __launch_bounds__(NT * KS) void conv3_kernel(const GemmArgs a, const int ny0, const int max_mtiles0) {
    int ny = ny0, max_mtiles = max_mtiles0;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int share = KS > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x / NT) : 0;
    char* As = smem + share * main_bytes(KS);          // [RMAX + 1][32] bf16
    char* Bs = As + A_BYTES;                           // [TPP][BN][32] bf16
    long long* rowC = (long long*)(smem + KS * main_bytes(KS));
    long long* rowR = rowC + BM;
    float* scl = (float*)(rowR + BM);                  // [BN] scale, then [BN] shift
    constexpr uint32_t OOB = 0x80000000u;

    const GroupLanes lanes(a.gt);
    const bf16_t *A = a.A, *Wt = a.Wt, *res = a.R;
    bf16_t* C = (bf16_t*)a.C;
    const float *scale = a.scale, *shift = a.shift;
    const int32_t *a_index = a.a_index, *c_index = a.c_index;
    int64_t a_ss = a.a_sample_stride, c_ss = a.c_sample_stride, r_ss = a.r_sample_stride;
    int a_ld = a.a_ld, c_ld = a.c_ld, r_ld = a.r_ld, c_row0 = a.c_row0, r_use = a.r_use_index, w_ld = (int)a.w_ld;
    int w_tap = (int)a.w_tap_stride, tab_ld = a.tab_ld, W = a.W, H = a.H, rows = a.rows, act = a.act;
    TileSource source(a);
    source.hold();
    ds_hold(A, Wt, res, C, scale, shift, a_index, c_index, a_ss, c_ss, r_ss, a_ld, c_ld, r_ld, c_row0, r_use, w_ld, w_tap, tab_ld, W, H,
            rows, act, ny, max_mtiles);
    const int j = (int)(blockIdx.x >> 3);
    const int jm = ds_quotient_uniform(j, ny), y = j - jm * ny;
    const int mt = jm * 8 + (int)(blockIdx.x & 7);
    if (mt >= max_mtiles) return;
    const int4 me = source.record(mt);
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

    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, l32 = lane & 31, lhi = lane >> 5;
    // ---- patch loader: item e = tid + 256 i is chunk (e & 3) of patch row (e >> 2).  A wavefront loads 64 rows, 16 of every 64: a lane works
    // out one of them, the lanes that load it get its address from there -------------------------------------------------------------
    static_assert(NR == 4, "a patch row per lane");
    const int lchunk = tid & 3;
    uint32_t poff[NR];
    {
        const int jr = 16 * wave + (lane & 15) + 64 * (lane >> 4);
        const int L = grow0 - halo + jr;              // pixel index in the group's row-major order
        uint32_t o = OOB;
        if (jr < R && L >= 0 && L < rows_g) {
            const int sl = ds_quotient(L, rows);
            const int p = L - sl * rows;
            const int slot = slot0 + sl;
            const int sa = a_index ? a_index[slot] : slot;
            o = (uint32_t)(((long long)sa * a_ss + (long long)p * a_ld) * 2);
        }
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            const uint32_t q = (uint32_t)__shfl((int)o, (lane >> 2) + 16 * i, 64);
            poff[i] = q == OOB ? OOB : q + lchunk * 16;
        }
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

    // ---- this lane's output pixel: where it goes, which taps are inside the image ---------------------------
    const int trow = wave * 32 + l32;
    int tapmask = 0;
    {
        const int m = grow0 + trow;
        long long rc = -1, rr = 0;
        if (m < rows_g) {
            const int sl = ds_quotient(m, rows);
            const int p = m - sl * rows;
            const int slot = slot0 + sl;
            const int cs = c_index ? c_index[slot] : slot;
            rc = (long long)cs * c_ss + (long long)(p + c_row0) * c_ld;
            rr = (long long)(r_use ? cs : 0) * r_ss + (long long)(p + c_row0) * r_ld;
            const int oy = ds_quotient(p, W), ox = p - oy * W;
            // filter columns, filter rows inside the map
            const int cols = (ox > 0 ? 1 : 0) | 2 | (ox + 1 < W ? 4 : 0);
            tapmask = (oy > 0 ? cols : 0) | cols << 3 | (oy + 1 < H ? cols << 6 : 0);
        }
        if (lane < 32 && share == 0) {
            rowC[trow] = rc;
            if constexpr (HASR) rowR[trow] = rr;
        }
    }

    f32x16_t acc[2];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[t][v] = 0.f;

    // epilogue constants and residual rows, fetched early so that their latency hides behind the loop
    if (threadIdx.x < BN) {
        const int n = n0 + tid;
        float vs = 1.f, vh = 0.f;
        if (n < k_out) {
            const long long ti = (long long)lanes.row(g) * tab_ld + n;
            if (scale) vs = scale[ti];
            if (shift) vh = shift[ti];
        }
        scl[tid] = vs;
        scl[BN + tid] = vh;
    }
    // One share: 8 channels of rows (lane / 8) + 8 i of the wavefront's 32; several: 4 channels of every 16 KS-th row of the tile.
    constexpr int NE = KS == 1 ? 4 : BM / (16 * KS);
    const int srow = lane >> 3, ncol8 = n0 + (lane & 7) * 8, ncol4 = n0 + ((int)threadIdx.x & 15) * 4;
    using Piece = typename std::conditional<KS == 1, uint4, uint2>::type;
    Piece rres[HASR ? NE : 1];
    if constexpr (HASR) {
        if constexpr (KS > 1) __syncthreads();         // row table visible
        else wave_sync();                              // (a wavefront's own rows)
#pragma unroll
        for (int i = 0; i < NE; ++i) {
            const int r = KS == 1 ? wave * 32 + srow + 8 * i : ((int)threadIdx.x >> 4) + i * 16 * KS;
            const int n = KS == 1 ? ncol8 : ncol4;
            Piece t = {};
            if (n < k_out && rowC[r] >= 0) t = *(const Piece*)(res + rowR[r] + n);
            rres[i] = t;
        }
    }

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
                for (int t = 0; t < 2; ++t) acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[t], af, acc[t], 0, 0, 0);
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

    // Filters are the instruction's row operand: a lane holds channels 32 tn + 8 q + 4 lhi .. + 3 of row l32 (gemm_kernel's epilogue)
    if constexpr (KS > 1) {
        // ---- partial tiles to LDS, added in share order (the loop's last barrier has retired every read of the slabs they take the place of)
        float* part = (float*)As;
#pragma unroll
        for (int tn = 0; tn < 2; ++tn)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *(float4*)(part + trow * PT_LD + tn * 32 + 8 * q + 4 * lhi) =
                    make_float4(acc[tn][4 * q], acc[tn][4 * q + 1], acc[tn][4 * q + 2], acc[tn][4 * q + 3]);
        __syncthreads();
        const int cg = threadIdx.x & 15;
        const float4 s4 = *(const float4*)(scl + cg * 4), h4 = *(const float4*)(scl + BN + cg * 4);
        with_act<false>(act, [&](auto actc) {
            constexpr int ACT = decltype(actc)::value;
#pragma unroll
            for (int i = 0; i < NE; ++i) {
                const int r = ((int)threadIdx.x >> 4) + i * 16 * KS;
                const long long coff = rowC[r];
                if (ncol4 >= k_out || coff < 0) continue;
                float4 t = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
                for (int k = 0; k < KS; ++k) {
                    const float4 p = *(const float4*)((const float*)(smem + k * main_bytes(KS)) + r * PT_LD + cg * 4);
                    t.x += p.x; t.y += p.y; t.z += p.z; t.w += p.w;
                }
                float val[4] = {t.x * s4.x + h4.x, t.y * s4.y + h4.y, t.z * s4.z + h4.z, t.w * s4.w + h4.w};
                if constexpr (HASR) add_residual(val, make_uint2(rres[i].x, rres[i].y));
                *(uint2*)(C + coff + ncol4) = activate_bf16<ACT>(val);
            }
        });
    } else {
        // ---- a wavefront's 32 x 64 tile through LDS as bf16, a residual parked there beforehand; it leaves as 16-byte pieces.  The stage is
        // private to a wavefront and the loop's last barrier has retired every read of the tiles it aliases
        bf16_t* st = (bf16_t*)smem + wave * 32 * ST_LD;
        if constexpr (HASR) {
#pragma unroll
            for (int i = 0; i < 4; ++i) *(Piece*)(st + (srow + 8 * i) * ST_LD + (lane & 7) * 8) = rres[i];
            wave_sync();
        }
        with_act<false>(act, [&](auto actc) {
            constexpr int ACT = decltype(actc)::value;
#pragma unroll
            for (int tn = 0; tn < 2; ++tn)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int ch = tn * 32 + 8 * q + 4 * lhi;
                    const float4 s4 = *(const float4*)(scl + ch), h4 = *(const float4*)(scl + BN + ch);
                    const f32x16_t& t = acc[tn];
                    float val[4] = {t[4 * q] * s4.x + h4.x, t[4 * q + 1] * s4.y + h4.y, t[4 * q + 2] * s4.z + h4.z, t[4 * q + 3] * s4.w + h4.w};
                    uint2* p = (uint2*)(st + l32 * ST_LD + ch);
                    if constexpr (HASR) add_residual(val, *p);
                    *p = activate_bf16<ACT>(val);
                }
        });
        wave_sync();
        if (ncol8 < k_out) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const long long coff = rowC[wave * 32 + srow + 8 * i];
                if (coff >= 0) *(uint4*)(C + coff + ncol8) = *(const uint4*)(st + (srow + 8 * i) * ST_LD + (lane & 7) * 8);
            }
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

// 3x3, stride 1, padding 1, one segment, bf16 results without GELU, maps up to 59 pixels wide; DS_EUNSUPPORTED otherwise
int32_t ds_launch_conv3(const GemmArgs& a, int32_t max_mtiles, int32_t max_kout, hipStream_t s) {
    if (a.K != 3 || a.stride != 1 || a.pad != 1 || a.n_seg != 1 || a.Ho != a.H || a.Wo != a.W || a.rows != a.H * a.W ||
        BM + 2 * (a.W + 1) > RMAX || !conv_result(a))
        return DS_EUNSUPPORTED;
    if (((long long)max_kout * a.w_ld + 9 * a.w_tap_stride) * 2 >= 0x7fffffffLL) return DS_EUNSUPPORTED;   // 32-bit weight offsets
    int kmax = 0;
    for (int t = 0; t < a.gt.T; ++t) kmax = a.gt.k_in[t] > kmax ? a.gt.k_in[t] : kmax;
    const int64_t wgs = (int64_t)max_mtiles * ((max_kout + BN - 1) / BN) * (a.crowd > 1 ? a.crowd : 1);
    // Shares of the reduction.  A workgroup is a chain of 3 phases a chunk, about 0.9 us each, whatever else runs; with fewer
    // workgroups than the compute units could hold, shares shorten it.  DS-ResNet, us a pass, one share -> here: 16 / 33 / 64 / 96 images 609 / 789 /
    // 1059 / 1245 -> 601 / 737 / 1006 / 1217, DS-ResNet++ 33 / 64 images 838 / 1165 -> 793 / 1109.  Half and twice these lines: 33 / 64 / 96 images 765 /
    // 1063 / 1243 and 746 / 1034 / 1203 (the shares of a workgroup wait for each other); four shares of 16 chunks up to 256 workgroups in place of 512: 64 /
    // 96 images 1011 / 1222.  Parts of a batch that run side by side count together: 256 images in four parts took 2894 us, 3097 with shares.
    const int ks = kmax > 64 && wgs <= (kmax > 256 ? 512 : 256) ? 4 : kmax > 32 && wgs <= 512 ? 2 : 1;
#define DS_CONV3(KS) (a.R ? launch<true, KS>(a, max_mtiles, max_kout, s) : launch<false, KS>(a, max_mtiles, max_kout, s))
    return ks == 4 ? DS_CONV3(4) : ks == 2 ? DS_CONV3(2) : DS_CONV3(1);
#undef DS_CONV3
}
