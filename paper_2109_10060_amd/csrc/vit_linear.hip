// Linear layers of a transformer block over tiled weights: rows stay in LDS, weights stream into registers.
//
//   y = act(LN(x) W^T + b) [+ residual], LayerNorm optional, up to three stacked segments (Q, K, V)
//
// A workgroup owns BM = 32 R token rows (whole rows: the LayerNorm is computed in place, the arithmetic of
// layernorm16_kernel) and a run of 32-column blocks of the output, NW at a time, one per wavefront.  A wavefront reads its
// weight operands as contiguous kilobytes straight into registers, D in flight, so neither the weights nor the partial
// sums touch LDS.  Two uses.
// Large batches: the first block's Q/K/V layer (the others come with the block in front, from a few dozen tiles on) with 8
// wavefronts and 64 rows, all columns in one workgroup (the rows are read once;
// gemm_kernel read them once per 64 columns).  A finished block is traded between the halves of the wavefront and stored from
// its registers, 16 bytes a lane (DIRECT): pieces of 64 bytes where a stage in LDS would make whole lines, but without the stage
// two workgroups share a compute unit, one normalises rows while the other multiplies, and no wavefront waits for another
// between blocks.  Us a pass, 12 wavefronts, 64 rows and a stage -> here: DS-ViT 64 / 140 / 256 images 880 / 1398 / 2284 -> 879 / 1391 / 2277,
// DS-ViT++ 1222 / 2142 / 3610 -> 1223 / 2135 / 3565.  (In every block, before the block in front brought Q/K/V: DS-ViT 1058 / 1697 / 2663
// -> 1041 / 1657 / 2643, DS-ViT++ 64 and 256 images 1418 / 3947 -> 1396 / 3801; eight operands in flight instead of four 3760, but the
// others 1049, 1681, 2652 and 1399; 32 rows 256 images 2700 and 3906.)
// Few images: all four layers of a block on 32 rows, where a launch is bound by latency and by how many compute units share the
// weights' way in: runs of four or eight column blocks with 4 wavefronts, or with 8 that fetch and normalise half as many rows each
// while four of them multiply, and two blocks a workgroup with 8 wavefronts in fc2, whose rows are the longest.  Finished blocks leave
// through an LDS tile as 16-byte pieces of whole row runs.  The LayerNorm launches disappear.  A LayerNorm there is a chain in front of
// the products: rows, then its weights (through LDS) and the first operands are asked for together, and its sums run over rotations
// within 16 lanes instead of exchanges through LDS.
// Sums are in gemm_kernel's order: the same bits.
#include "gelu.h"
#include "vit_rows.h"
#include "vit_run.h"

namespace {

// KM: channels of the reduction, at most.  DIRECT: stores from registers (no residual, no activation).  FEW: a launch of a few images, a chain of latencies: everything asked for as early as it can be
template <int NW, int R, int D, int KM, bool FEW, bool DIRECT>
__global__ __launch_bounds__(64 * NW, DIRECT ? NW / 2 : (NW + 3) / 4) void vit_linear_kernel(const VitLinearArgs a, const int runs, const int run_blocks) {
    constexpr int PITCH = tile_pitch(KM, D);
    constexpr int BM = 32 * R, SP = 32 * NW + 8, RP = 4 * NW, NI = (BM + RP - 1) / RP, KIT = (PITCH - 8 + 127) / 128, NS = 4 * NW;
    extern __shared__ __attribute__((aligned(16))) char smem[];
    bf16_t* As = (bf16_t*)smem;                          // [BM][PITCH]
    bf16_t* Ss = As + BM * PITCH;                        // [BM][SP] output stage

    const int tile = ds_quotient_uniform((int)blockIdx.x, runs), run = (int)blockIdx.x - tile * runs;
    const GroupLanes lanes(a.gt);
    const bf16_t *x = a.x, *wt = a.w, *res = a.res;
    bf16_t* y = a.y;
    const float *gamma = a.gamma, *beta = a.beta, *bias0 = a.bias;
    int64_t x_ss = a.x_ss, y_ss = a.y_ss, y_seg = a.y_seg;
    int x_ld = a.x_ld, y_ld = a.y_ld, rows = a.rows, kb = a.kb, seg_blocks = a.seg_blocks, n_seg = a.n_seg, bias_seg = a.bias_seg, act = a.act;
    float eps = a.eps;
    const int4 me = ds_tile_record_of(a.offsets, a.gt.T, rows, tile, BM);
    if constexpr (FEW)
        ds_hold(x, wt, res, y, gamma, beta, bias0, x_ss, y_ss, y_seg, x_ld, y_ld, rows, kb, seg_blocks, n_seg, bias_seg, act, eps);
    if (me.x < 0) return;
    const int g = me.x, grow0 = me.y, slot0 = me.z, rows_g = me.w;
    const int kin = lanes.k_in(g), k_out = lanes.k_out(g);
    if (kin <= 0 || k_out <= 0) return;
    const int nb = (k_out + 31) / 32, total = nb * n_seg;      // column blocks of a segment, of the layer
    const int blk0 = run * run_blocks, blk1 = min(total, blk0 + run_blocks);
    if (blk0 >= total) return;

    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, l32 = lane & 31, lhi = lane >> 5;
    const int l16 = tid & 15, prow = tid >> 4;
    const uint32_t lane16 = (uint32_t)lane * 16;
    if (x_ld <= 0) x_ld = kin;
    if (y_ld <= 0) y_ld = k_out;

    bf16x8_t ring[D];
    auto weights = [&](int p) {
        const int s = run_segment(p, nb);
        return weight_row(wt, (s * seg_blocks + p - s * nb) * kb, kin);
    };
    auto start = [&](int p, bool on = true) {            // (off: no traffic)
        const __amdgpu_buffer_rsrc_t rw = on ? weights(p) : weight_row(wt, 0, 0);
#pragma unroll
        for (int j = 0; j < D; ++j) ring[j] = weight_tile(rw, lane16 + j * 1024);
    };
    if (!FEW && blk0 + w < blk1) start(blk0 + w);        // the weights are under way while the rows are fetched

    // ---- rows -------------------------------------------------------------------------------------------------------------
    int64_t yoff[NI];
    bool live[NI];
    uint4 q[NI][KIT];
    auto fetch_rows = [&](int i) {
        const bool in = BM % RP == 0 || prow + RP * i < BM;
        const int m = grow0 + prow + RP * i;
        live[i] = in && m < rows_g;
        const int mm = live[i] ? m : grow0;
        const int sl = ds_quotient(mm, rows), p = mm - sl * rows, slot = slot0 + sl;
        yoff[i] = (int64_t)slot * y_ss + (int64_t)p * y_ld;
        const bf16_t* xrow = x + (int64_t)slot * x_ss + (int64_t)p * x_ld;
#pragma unroll
        for (int k = 0; k < KIT; ++k) {
            const int ch = (k * 16 + l16) * 8;
            if constexpr (FEW) {
                q[i][k] = *(const uint4*)(xrow + (ch < kin ? ch : 0));       // no branch around a request: see below
            } else {
                q[i][k] = make_uint4(0, 0, 0, 0);
                if (ch < kin) q[i][k] = *(const uint4*)(xrow + ch);
            }
        }
    };
    constexpr bool NORM = KM <= VIT_K_MAX;
    constexpr bool SKIP = !DIRECT && !(FEW && NW == 8);  // (row_stats)
    constexpr int KN = KIT < 4 ? KIT : 4;                // 16-byte chunks of a lane inside the widest slice
    float* gs = (float*)(Ss + BM * SP);                  // (FEW) LayerNorm weights: gamma, then beta
    if constexpr (FEW) {
        // Loads return in order, so what a wavefront needs first is asked for first: its rows, the LayerNorm weights (a share of them each,
        // through LDS: read by every wavefront for itself they were 16 KiB each ahead of the rows), then the operands of the first products.
        // Rows and operands without a branch around them: behind one the number in flight is not known, and the rows would wait for
        // the operands as well.
#pragma unroll
        for (int i = 0; i < NI; ++i) fetch_rows(i);
        if constexpr (NORM) {
            if (gamma)
                for (int c = tid * 4; c < kin; c += 64 * NW * 4) {
                    *(float4*)(gs + c) = *(const float4*)(gamma + c);
                    *(float4*)(gs + VIT_K_MAX + c) = *(const float4*)(beta + c);
                }
        }
        start(blk0 + w, blk0 + w < blk1);
        if constexpr (NORM) {
            if (gamma) __syncthreads();
        }
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int k = 0; k < KIT; ++k)
            {
                const uint32_t keep = (k * 16 + l16) * 8 < kin ? ~0u : 0u;
                q[i][k] = make_uint4(q[i][k].x & keep, q[i][k].y & keep, q[i][k].z & keep, q[i][k].w & keep);
            }
    }
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        if constexpr (!FEW) fetch_rows(i);
        const bool in = BM % RP == 0 || prow + RP * i < BM;
        if constexpr (NORM) {
            if (gamma) {
                float v[4][8];
                uint4 o[4];
#pragma unroll
                for (int k = 0; k < KN; ++k)
                    if (row_has<SKIP>(k, kin)) unpack8(q[i][k], v[k]);
                if constexpr (FEW) row_norm<SKIP>(v, kin, l16, eps, gs, gs + VIT_K_MAX, o);
                else row_norm<SKIP>(v, kin, l16, eps, gamma, beta, o);
#pragma unroll
                for (int k = 0; k < KN; ++k)
                    if ((k * 16 + l16) * 8 < kin) q[i][k] = o[k];
            }
        }
#pragma unroll
        for (int k = 0; k < KIT; ++k) {
            const int ch = (k * 16 + l16) * 8;
            if (in && ch < PITCH) *(uint4*)(As + (prow + RP * i) * PITCH + ch) = q[i][k];     // zeros beyond the slice
        }
    }

    // the products of column block p; every step is straight-line code, the operands of the next one on their way
    auto walk = [&](f32x16_t (&acc)[R], int p) __attribute__((always_inline)) {
        const __amdgpu_buffer_rsrc_t rw = weights(p);
        const bf16_t* base = As + l32 * PITCH + lhi * 8;
        bf16x8_t f[2][R];
#pragma unroll
        for (int r = 0; r < R; ++r) f[0][r] = *(const bf16x8_t*)(base + r * 32 * PITCH);
        uint32_t off = lane16 + D * 1024;
        for (int k0 = 0; k0 < kin; k0 += 16 * D, off += D * 1024) {       // rounded up to D: zero weights, zeros behind the slice (tile_pitch)
#pragma unroll
            for (int j = 0; j < D; ++j) {
#pragma unroll
                for (int r = 0; r < R; ++r) f[(j + 1) & 1][r] = *(const bf16x8_t*)(base + r * 32 * PITCH + k0 + (j + 1) * 16);
#pragma unroll
                for (int r = 0; r < R; ++r) acc[r] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[j], f[j & 1][r], acc[r], 0, 0, 0);
                ring[j] = weight_tile(rw, off + j * 1024);
                __builtin_amdgcn_sched_barrier(0);       // (the compiler would sink the reads to their use)
            }
        }
    };
    auto clear = [](f32x16_t (&acc)[R]) {
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[r][v] = 0.f;
    };
    if constexpr (DIRECT) {
        // ---- column blocks, each wavefront its own: no stage, so no wavefront waits for another ----
        __syncthreads();
        bf16_t* yrow[R];
        bool in[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int m = grow0 + r * 32 + l32;
            in[r] = m < rows_g;
            const int mm = in[r] ? m : grow0, sl = ds_quotient(mm, rows);
            yrow[r] = y + (int64_t)(slot0 + sl) * y_ss + (int64_t)(mm - sl * rows) * y_ld;
        }
        for (int p = blk0 + w; p < blk1; p += NW) {
            const int seg = run_segment(p, nb), n0 = (p - seg * nb) * 32;
            f32x16_t acc[R];
            clear(acc);
            walk(acc, p);
            if (p + NW < blk1) start(p + NW);
            const float* bias = bias0 + (int64_t)seg * bias_seg;
            const int64_t so = (int64_t)seg * y_seg;
#pragma unroll
            for (int q = 0; q < 4; q += 2) {
                float4 h[2];
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const int n = n0 + 8 * (q + e) + 4 * lhi;
                    h[e] = n < k_out ? *(const float4*)(bias + n) : make_float4(0.f, 0.f, 0.f, 0.f);
                }
                const int n = n0 + 8 * q + 8 * lhi;
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    uint32_t lo[2], hi[2];
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        const f32x16_t& t = acc[r];
                        const int b = 4 * (q + e);
                        lo[e] = f2bf2(t[b] + h[e].x, t[b + 1] + h[e].y);
                        hi[e] = f2bf2(t[b + 2] + h[e].z, t[b + 3] + h[e].w);
                    }
                    // channels 8 q .. + 7 to the lower half's lane, the next eight to the upper half's
                    const auto a0 = __builtin_amdgcn_permlane32_swap(lo[0], lo[1], false, false);
                    const auto a1 = __builtin_amdgcn_permlane32_swap(hi[0], hi[1], false, false);
                    if (in[r] && n < k_out) *(uint4*)(yrow[r] + so + n) = make_uint4(a0[0], a1[0], a0[1], a1[1]);
                }
            }
        }
        return;
    }
    // ---- column blocks, NW at a time ------------------------------------------------------------------------------------------
    for (int b0 = blk0; b0 < blk1; b0 += NW) {
        const int p = b0 + w, seg = run_segment(p, nb), n0 = (p - seg * nb) * 32;
        const bool on = p < blk1;
        if (res) {
            // the residual of these columns waits in the stage, where the sums are added in place; this run's columns only: res may be
            // y, and the next workgroup's columns are being written
#pragma unroll
            for (int i = 0; i < NI; ++i)
#pragma unroll
                for (int k = 0; k < (NS + 15) / 16; ++k) {
                    const int c = k * 16 + l16, n = (b0 + (c >> 2)) * 32 + (c & 3) * 8;
                    if (run_chunk(c, NW, b0, blk1) && live[i] && n < k_out)
                        *(uint4*)(Ss + (prow + RP * i) * SP + c * 8) = *(const uint4*)(res + yoff[i] + n);
                }
        }
        __syncthreads();                                 // rows (and residual) are in place
        f32x16_t acc[R];
        clear(acc);
        if (on) {
            const float* bias = bias0 + (int64_t)seg * bias_seg;
            float4 hb[FEW ? 4 : 1];
            if constexpr (FEW) {
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int n = n0 + 8 * q + 4 * lhi;
                    hb[q] = n < k_out ? *(const float4*)(bias + n) : make_float4(0.f, 0.f, 0.f, 0.f);
                }
            }
            walk(acc, p);
            if (p + NW < blk1) start(p + NW);
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int n = n0 + 8 * q + 4 * lhi;
                if (n >= k_out) continue;
                const float4 h = FEW ? hb[FEW ? q : 0] : *(const float4*)(bias + n);
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    uint2* s = (uint2*)(Ss + (r * 32 + l32) * SP + w * 32 + 8 * q + 4 * lhi);
                    float v0 = acc[r][4 * q] + h.x, v1 = acc[r][4 * q + 1] + h.y, v2 = acc[r][4 * q + 2] + h.z, v3 = acc[r][4 * q + 3] + h.w;
                    if (act == DS_ACT_GELU) {
                        *s = gelu_bf16x4(v0, v1, v2, v3);
                        continue;
                    }
                    if (res) {
                        const uint2 t = *s;
                        v0 += __uint_as_float(t.x << 16);
                        v1 += __uint_as_float(t.x & 0xffff0000u);
                        v2 += __uint_as_float(t.y << 16);
                        v3 += __uint_as_float(t.y & 0xffff0000u);
                    }
                    *s = make_uint2(f2bf2(v0, v1), f2bf2(v2, v3));
                }
            }
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int k = 0; k < (NS + 15) / 16; ++k) {
                const int c = k * 16 + l16, pb = b0 + (c >> 2);
                if (!run_chunk(c, NW, b0, blk1) || !live[i]) continue;
                const int sg = run_segment(pb, nb), n = (pb - sg * nb) * 32 + (c & 3) * 8;
                if (n < k_out) *(uint4*)(y + yoff[i] + (int64_t)sg * y_seg + n) = *(const uint4*)(Ss + (prow + RP * i) * SP + c * 8);
            }
        if (b0 + NW < blk1) __syncthreads();             // the stage is free again
    }
}

template <int NW, int R, int D, int KM, bool FEW, bool DIRECT = false>
int32_t launch(const VitLinearArgs& a, int64_t tiles, int max_blocks, int run_blocks, hipStream_t s) {
    constexpr int SMEM = 32 * R * (tile_pitch(KM, D) + (DIRECT ? 0 : 32 * NW + 8)) * 2 + (DIRECT ? 32 : 0) + (FEW && KM <= VIT_K_MAX ? 2 * VIT_K_MAX * 4 : 0);
    static_assert(SMEM <= 160 * 1024, "LDS of a compute unit");
    const int32_t rc = ds_reserve_lds((const void*)vit_linear_kernel<NW, R, D, KM, FEW, DIRECT>, SMEM, "tiled linear layer");
    if (rc) return rc;
    const int runs = (max_blocks + run_blocks - 1) / run_blocks;
    ProfScope prof(DS_K_VIT_LINEAR, s);
    hipLaunchKernelGGL((vit_linear_kernel<NW, R, D, KM, FEW, DIRECT>), dim3((unsigned)(tiles * runs)), dim3(64 * NW), SMEM, s, a, runs, run_blocks);
    DS_CHECK_LAUNCH("tiled linear layer");
    return DS_OK;
}

}  // namespace

// Column blocks a workgroup, us a pass (profiles/dispatch_choices.txt), four / eight: DS-ViT 1 / 5 / 8 images 398 / 487 / 484 and 504 / 550 / 502, 12 / 16
// images 600 / 578 and 598 / 576; DS-ViT++ 7 / 9 images 682 / 905 and 726 / 931, 12 / 18 images 961 / 1002 and 937 / 965.  From 160 tiles of 64 rows on the
// large form, which is then the first block's alone: a pass of DS-ViT of 32 / 40 / 50 / 60 images, the line at 100 tiles 666 / 678 / 785 / 860, at 160
// 666 / 678 / 784 / 862, at 260 667 / 681 / 789 / 869; DS-ViT++ 40 / 60 / 66 images 1066 / 1189 / 1262, 1067 / 1190 / 1263, 1066 / 1193 / 1270.
// Reductions beyond 416 channels (fc2) are for the few-image path alone: 113 KiB of rows.  Us a pass, 4 wavefronts and four blocks a workgroup / 8 and
// two: DS-ViT 1 / 3 / 5 images 404 / 437 / 490 and 399 / 432 / 487, DS-ViT++ 1 / 5 images 489 / 618 and 484 / 616.
int32_t ds_launch_vit_linear(const VitLinearArgs& a, int32_t B, hipStream_t s) {
    int kmax = 0, nmax = 0;
    for (int t = 0; t < a.gt.T; ++t) {
        kmax = a.gt.k_in[t] > kmax ? a.gt.k_in[t] : kmax;
        nmax = a.gt.k_out[t] > nmax ? a.gt.k_out[t] : nmax;
        if ((a.gt.k_in[t] % 8) || (a.gt.k_out[t] % 8)) return DS_EUNSUPPORTED;
    }
    if (kmax <= 0 || nmax <= 0) return DS_OK;
    if ((a.n_seg > 1 && a.res) || a.n_seg > RUN_SEGMENTS) return DS_EUNSUPPORTED;
    const int64_t groups = B < a.gt.T ? B : a.gt.T, n = (int64_t)B * a.rows;
    auto tiles = [&](int bm) { return (n - groups) / bm + groups; };
    const int blocks = (nmax + 31) / 32 * a.n_seg;
    if (kmax <= VIT_K_MAX) {
        if (!a.res && a.act == DS_ACT_NONE && tiles(64) >= 160) {
            // parts of a batch, each with a workgroup a compute unit at most: two small ones would share the compute units that the other
            // part leaves free.  Us a pass, 8 / 12 wavefronts: DS-ViT in two parts, 96 images 1028 / 1021, 128 images 1225 / 1210, 160 images (293
            // tiles a part) 1488 / 1485, 200 images 1808 / 1792, 200 in four (219 tiles) 1838 / 1842; DS-ViT++ in two, 96 / 128 images 1562 / 1559, 1809 / 1803
            if (a.crowd > 1 && tiles(64) <= 256) return launch<12, 2, 4, VIT_K_MAX, false>(a, tiles(64), blocks, blocks, s);
            return launch<8, 2, 4, VIT_K_MAX, false, true>(a, tiles(64), blocks, blocks, s);
        }
        // (everything asked for early takes 10 registers more, 170 for 160, and with them the third workgroup of a compute unit.  Us a pass,
        // never early / here: DS-ViT 5 / 7 / 8 / 12 / 16 images 513 / 528 / 496 / 600 / 578 and 486 / 502 / 484 / 598 / 576, DS-ViT++ 5 / 9 / 12 / 18 images, where
        // every block has one, 653 / 931 / 962 / 999 and 614 / 905 / 936 / 964.  Beyond 128 tiles no batch differs; beside the launches of a batch's
        // other parts 32 / 48 / 64 images of DS-ViT in four 699 / 733 / 870 without, 703 / 731 / 869 with)
        const int run = tiles(32) > 64 ? 8 : 4;
        // up to a workgroup a compute unit eight wavefronts: half as many rows each to fetch and normalise, four of them multiply
        // (1 / 3 / 5 images 494 / 535 / 562 -> 474 / 515 / 558 us a pass when a wavefront asked for its LayerNorm weights itself; since they come
        // through LDS, up to two for some compute units measure better: 5 / 7 images 486 / 502 and 467 / 491, DS-ViT++ 614 / 681 and 586 / 667)
        if (a.crowd <= 1 && run == 4 && tiles(32) * ((blocks + 3) / 4) <= 256)
            return launch<8, 1, 8, VIT_K_MAX, true>(a, tiles(32), blocks, run, s);
        if (a.crowd <= 1 && tiles(32) <= 128) return launch<4, 1, 8, VIT_K_MAX, true>(a, tiles(32), blocks, run, s);
        return launch<4, 1, 8, VIT_K_MAX, false>(a, tiles(32), blocks, run, s);
    }
    if (kmax > 1664 || a.gamma) return DS_EUNSUPPORTED;
    // (a workgroup has its compute unit to itself: where runs of two column blocks would fill the chip, four.  Us a pass, two / four: DS-ViT 3 / 5
    // images 432 / 487 and 433 / 487, 6 / 7 images (252 and 294 workgroups of two) 505 / 540 and 499 / 504, 7 on the widest route 668 and 584; DS-ViT++
    // 3 / 5 images (245) 552 / 616 and 556 / 616, 7 images 723 and 681, 6 on the widest route 781 and 673)
    return launch<8, 1, 16, 1664, true>(a, tiles(32), blocks, tiles(32) * ((blocks + 1) / 2) <= 224 ? 2 : 4, s);
}
