// Grouped prefix-slice GEMM / implicit-GEMM convolution on the gfx950 matrix cores.
//
// One launch serves every route group of a layer.  Group g owns a contiguous
// range of bucket slots and multiplies its rows by the leading block
// W[:k_out[g], :k_in[g]] of the stored weight, read in place through the
// full-size leading stride (weight slicing, Section 3.2 Eq. 8; convolution
// filters, Section 3.3 Eq. 9).  A row of a sample is one token (linear layers)
// or one output pixel of a KxK convolution over an NHWC image; in the second
// case the K*K taps are walked inside the reduction loop and the A operand is
// gathered from the shifted input pixels (zero outside the image).
//
// Tiling: 128 x 64 output tile per 256-thread workgroup, 4 wavefronts, each holding a 32 x 64 grid of
// v_mfma_f32_32x32x16_bf16 accumulators (the dispatcher uses this shape for nearly every layer: with ragged route
// groups and slices as narrow as 64 channels the wider 128 x 128 / 128 x 256 instantiations lose more to
// quantisation and residency than their lower operand traffic gains).  Operands go through one LDS tile in
// 32-deep slabs, 64-deep ones for reductions of 256 steps and more, or 128-deep ones where a launch is about one
// generation of workgroups and a filter tap has 512 channels or more (the last ResNet stage: half as many dependent
// load -> LDS -> barrier rounds per workgroup; 64-, 128- or 256-byte rows, 16-byte chunks XOR-swizzled by row so
// stores and reads are bank-conflict free); the next slab's global loads are issued into
// registers before the current slab's matrix instructions and stored to LDS after them, and four to seven resident
// workgroups per compute unit (residency) hide each other's round trips.  The epilogue (split batch-norm scale and
// shift or bias, residual, ReLU/GELU, bf16 rounding) passes a wavefront's tile through LDS as bf16, and it leaves as
// 16-byte pieces, eight lanes a row.
//
// Work items are (m-tile, n-tile) pairs with the n-tile fastest; the linear block
// index is dealt round-robin to the 8 XCDs by the hardware, so each XCD is given
// a contiguous run of work items and the blocks that share an activation tile hit
// the same L2.
#include "tile_out.h"

namespace {

constexpr int BM = DS_GEMM_BM, NT = 256;   // NT: threads of a share of the reduction

// 16-byte chunk c of LDS row r is stored at chunk position c ^ swz(r): rows are BK * 2 bytes with no
// padding; the row-major stores and the operand reads (32 consecutive rows, one chunk column) are
// bank-conflict free for 8- and 16-lane access groups alike
template <int BK>
__device__ __forceinline__ int swz(int r) {
    return BK == 128 ? (r & 15) : BK == 64 ? ((r ^ (r >> 3)) & 7) : (((r >> 1) ^ (r >> 2)) & 3);
}

template <int WROWS, int WCOLS, int WMT, int WNT, int BK, int KS>
struct Tile {
    static constexpr int BN = WCOLS * WNT * 32, LDS_LD = BK;
    static constexpr int COLS = WNT * 32;                      // columns staged per wavefront
    static constexpr int ST_LD = COLS + 8;                     // of the bf16 stage: an odd number of 16-byte chunks
    static constexpr int PT_LD = BN + 4;                       // of a share's partial tile (fp32)
    static constexpr int LOOP_BYTES = (BM + BN) * LDS_LD * 2;
    static constexpr int STAGE_BYTES = KS > 1 ? 0 : 4 * 32 * ST_LD * 2;
    static constexpr int PART_BYTES = KS > 1 ? BM * PT_LD * 4 : 0;
    static constexpr int MAIN0 = LOOP_BYTES > STAGE_BYTES ? LOOP_BYTES : STAGE_BYTES;
    static constexpr int MAIN_BYTES = MAIN0 > PART_BYTES ? MAIN0 : PART_BYTES;    // of a share
    static constexpr int TABLE_BYTES = BM * (8 + 8) + 2 * BN * 4;   // output and residual rows, scale / shift of the tile's columns
    static constexpr int SMEM = KS * MAIN_BYTES + TABLE_BYTES;
    static_assert(KS == 1 || (WCOLS == 1 && WMT == 1 && SMEM <= 160 * 1024), "");
    static_assert(WROWS * WCOLS == 4 && WROWS * WMT * 32 == BM, "4 wavefronts cover a 128-row tile");
};

// Two 1x1 layers of one input (a stage's first layer and its projection) as one launch: the first layer's workgroups, then the other's.
// Apart, each of them starts with empty compute units and ends with most of them idle, 7 to 9 us together, and neither waits for the
// other.  DS-ResNet, us a pass, two launches -> here: 33 images 750 -> 736, 64 images 1022 -> 1009, 96 images 1221 -> 1214, 256 images 2428 ->
// 2418; DS-ResNet++ 33 / 64 / 256 images 805 / 1124 / 2816 -> 793 / 1108 / 2800.  Only pairs of up to 4000 or 8000 workgroups, before tiles left
// as 16-byte pieces (96 images 1320 without a limit): 1340 and 1331, 256 images (2597) 2611 and 2605.
struct GemmPair {
    GemmArgs p[2];
    uint32_t split;                      // workgroups of the first layer
    int32_t ny[2], mtiles[2];
};
__device__ __forceinline__ unsigned layer_of(const GemmArgs&) { return 0; }
__device__ __forceinline__ unsigned layer_of(const GemmPair& p) { return blockIdx.x >= p.split; }
__device__ __forceinline__ const GemmArgs& args_of(const GemmArgs& a, unsigned) { return a; }
__device__ __forceinline__ const GemmArgs& args_of(const GemmPair& p, unsigned q) { return p.p[q]; }

// Wavefronts a SIMD that the registers have to leave room for.  The 32-deep slabs live on residency: left to itself the convolution form takes
// 104 registers, four wavefronts, where six fit in 80 without scratch (256 -> 512 channels, 1x1/2 on 56x56, 256 images 109.8 -> 95.2 us, 64
// images 28.7 -> 24.9).  The 128-column tile of the same slabs measures the same with three and with four (256 -> 128 channels, 142.3 and 142.7).
constexpr int residency(int tiles, int bk, int shares, bool conv, bool res) {
    if (shares > 1 || tiles == 4) return 1;
    if (bk == 128) return 3;
    if (bk == 32) return res ? (conv ? 1 : 5) : 6;
    return conv ? 1 : 5;
}

// KS: shares of the reduction, four wavefronts each; a share takes every KS-th slab.  F32: fp32 results, of linear layers (several shares
// look at the argument instead: their way out is the same but for the store)
template <int WROWS, int WCOLS, int WMT, int WNT, int BK, int KS, bool CONV, bool HASR, bool F32, class Args = GemmArgs>
__global__ __launch_bounds__(NT * KS, residency(WMT * WNT, BK, KS, CONV, HASR)) void gemm_kernel(const Args args, const int ny0, const int max_mtiles0) {
    constexpr bool PAIR = std::is_same<Args, GemmPair>::value;
    const unsigned q = layer_of(args);
    const GemmArgs& a = args_of(args, q);
    unsigned block = blockIdx.x;
    int ny = ny0, max_mtiles = max_mtiles0;
    if constexpr (PAIR) {
        if (q) block -= args.split;
        ny = args.ny[q];
        max_mtiles = args.mtiles[q];
    }
    using TL = Tile<WROWS, WCOLS, WMT, WNT, BK, KS>;
    constexpr int BN = TL::BN, LDS_LD = BK, CPR = BK / 8, RPT = NT / CPR;   // chunks per row, rows per pass
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int share = KS > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x / NT) : 0;
    bf16_t* As = (bf16_t*)(smem + share * TL::MAIN_BYTES);   // [BM][BK]
    bf16_t* Bs = As + BM * LDS_LD;                    // [BN][BK]
    long long* rowC = (long long*)(smem + KS * TL::MAIN_BYTES);
    long long* rowR = rowC + BM;
    float* scl = (float*)(rowR + BM);                 // [BN] scale, then [BN] shift of this tile's output columns
    // operands are fetched with buffer loads: 32-bit byte offsets against a uniform base, and an
    // offset beyond the descriptor's range returns zeros, which supplies every tail (rows beyond
    // the group, channels beyond the slice, taps outside the image) without branches
    constexpr uint32_t OOB = 0x80000000u;

    // ---- work item ------------------------------------------------------------------
    // m-tiles are dealt to the 8 XCDs round-robin; on one XCD consecutive blocks walk the n-tiles
    // of one m-tile, so the activation tile they share stays in that XCD's L2
    const GroupLanes lanes(a.gt);
    const bf16_t *A = a.A, *Wt = a.Wt, *R = a.R;
    void* C = a.C;
    const float *scale = a.scale, *shift = a.shift;
    const int32_t *a_index = a.a_index, *c_index = a.c_index;
    int64_t a_ss = a.a_sample_stride, c_ss = a.c_sample_stride, r_ss = a.r_sample_stride, c_segs = a.c_seg_stride;
    int64_t w_ld = a.w_ld, w_tap = a.w_tap_stride, w_seg = a.w_seg_stride;
    int a_ld = a.a_ld, c_ld = a.c_ld, r_ld = a.r_ld, c_row0 = a.c_row0, r_use = a.r_use_index;
    int n_seg = a.n_seg, tab_ld = a.tab_ld, tab_seg = a.tab_seg_stride, rows = a.rows, act = a.act, out_f32 = KS > 1 && !CONV ? a.out_f32 : 0;
    int KH = a.K, KW = a.Kw, H = a.H, W = a.W, Wo = a.Wo, sy = a.stride, sx = a.stride_w, pad = a.pad;
    TileSource source(a);
    source.hold();
    ds_hold(ny, max_mtiles, A, Wt, R, C, scale, shift, a_index, c_index, a_ss, c_ss, r_ss, c_segs, w_ld, w_tap, w_seg, a_ld, c_ld, r_ld, c_row0, r_use,
            n_seg, tab_ld, tab_seg, rows, act, KH, KW);
    if constexpr (KS > 1 && !CONV) ds_hold(out_f32);
    if constexpr (CONV) ds_hold(H, W, Wo, sy, sx, pad);
    const int j = (int)(block >> 3);
    const int jm = ds_quotient_uniform(j, ny), y = j - jm * ny;
    const int mt = jm * 8 + (int)(block & 7);
    if (mt >= max_mtiles) return;
    const int4 me = source.record(mt);
    if (me.x < 0) return;
    const int g = me.x, grow0 = me.y, slot0 = me.z, rows_g = me.w;
    const int k_in = lanes.k_in(g), k_out = lanes.k_out(g);
    if (k_in <= 0 || k_out <= 0) return;
    int seg = 0, n0 = y * BN;
    if (n_seg > 1) {
        const int ntiles = (k_out + BN - 1) / BN;
        seg = y / ntiles;
        if (seg >= n_seg) return;
        n0 -= seg * ntiles * BN;
    }
    if (n0 >= k_out) return;

    const __amdgpu_buffer_rsrc_t rsrc_a = __builtin_amdgcn_make_buffer_rsrc((void*)A, 0, 0x7fffffff, 0x00020000);
    const __amdgpu_buffer_rsrc_t rsrc_w = __builtin_amdgcn_make_buffer_rsrc((void*)Wt, 0, 0x7fffffff, 0x00020000);
    const int tid = KS > 1 ? threadIdx.x & (NT - 1) : threadIdx.x;   // of the share
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int wm = wave / WCOLS, wn = wave - wm * WCOLS;
    const int l32 = lane & 31, lhi = lane >> 5;
    if (a_ld <= 0) a_ld = k_in;
    if (c_ld <= 0) c_ld = k_out;
    if (r_ld <= 0) r_ld = k_out;
    if (KW <= 0) KW = KH;
    if (sx <= 0) sx = sy;

    // ---- rows: a lane works out row l32 of the 32 its wavefront loads; the lanes that load a row get its address from that lane ------
    uint32_t my_a = OOB;
    int2 my_yx = make_int2(0, 0);
    {
        const int m = grow0 + 32 * wave + l32;
        long long rc = -1, rr = 0;
        if (m < rows_g) {
            const int sl = ds_quotient(m, rows);
            const int p = m - sl * rows;
            const int slot = slot0 + sl;
            const int sa = a_index ? a_index[slot] : slot;
            const int cs = c_index ? c_index[slot] : slot;
            // byte offset of the sample (convolution) or of the row itself (linear layers)
            my_a = (uint32_t)(((long long)sa * a_ss + (CONV ? 0 : (long long)p * a_ld)) * 2);
            if constexpr (CONV) {
                const int oy = ds_quotient(p, Wo), ox = p - oy * Wo;
                my_yx = make_int2(oy * sy - pad, ox * sx - pad);
            }
            const long long pc = p + c_row0;
            rc = (long long)cs * c_ss + pc * c_ld + (long long)seg * c_segs;
            rr = (long long)(r_use ? cs : 0) * r_ss + pc * r_ld;
        }
        if (lane < 32 && (KS == 1 || share == 0)) {           // read behind the loop's barriers
            rowC[32 * wave + l32] = rc;
            if constexpr (HASR) rowR[32 * wave + l32] = rr;
        }
    }

    // ---- load assignment: a lane owns chunk (lane % CPR) of rows (lane / CPR) + RPW i of its wavefront's 32, and of rows (tid / CPR) + RPT i of the weights
    constexpr int NA = BM / RPT, NB = BN / RPT, RPW = 64 / CPR;
    const int lchunk = tid % CPR;
    const int kc8 = lchunk * 8;
    const int lrow = tid / CPR, arow = lane / CPR;
    uint32_t aoff[NA], apix[NA], woff[NB];
    int2 ayx[CONV ? NA : 1];
#pragma unroll
    for (int i = 0; i < NA; ++i) {
        aoff[i] = (uint32_t)__shfl((int)my_a, arow + RPW * i, 64);
        if constexpr (CONV) ayx[i] = make_int2(__shfl(my_yx.x, arow + RPW * i, 64), __shfl(my_yx.y, arow + RPW * i, 64));
        apix[i] = aoff[i] == OOB ? OOB : aoff[i] + kc8 * 2;
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int n = n0 + lrow + RPT * i;
        woff[i] = n < k_out ? (uint32_t)(((long long)seg * w_seg + (long long)n * w_ld + kc8) * 2) : OOB;
    }
    // per filter tap: byte offset of the input pixel each owned row reads (OOB outside the image)
    auto set_tap = [&](int tap) {
        if constexpr (CONV) {
            const int u = tap / KW, v = tap - u * KW;
#pragma unroll
            for (int i = 0; i < NA; ++i) {
                const int iy = ayx[i].x + u, ix = ayx[i].y + v;
                const bool ok = aoff[i] != OOB && iy >= 0 && iy < H && ix >= 0 && ix < W;
                apix[i] = ok ? aoff[i] + (uint32_t)(((iy * W + ix) * a_ld + kc8) * 2) : OOB;
            }
        }
    };

    uint4 ra[NA], rb[NB];
    auto load_global = [&](int tap, int kc, bool on) {
        const bool kok = on && (kc + kc8) < k_in;
        const int soff_a = kc * 2;
        const int soff_w = (int)((tap * w_tap + kc) * 2);
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            const auto t = __builtin_amdgcn_raw_buffer_load_b128(rsrc_a, (int)(kok ? apix[i] : OOB), soff_a, 0);
            ra[i] = make_uint4(t[0], t[1], t[2], t[3]);
        }
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const auto t = __builtin_amdgcn_raw_buffer_load_b128(rsrc_w, (int)(kok ? woff[i] : OOB), soff_w, 0);
            rb[i] = make_uint4(t[0], t[1], t[2], t[3]);
        }
    };
    auto store_lds = [&]() {
#pragma unroll
        for (int i = 0; i < NA; ++i) {
            const int r = 32 * wave + arow + RPW * i;
            *(uint4*)(As + r * LDS_LD + ((lchunk ^ swz<BK>(r)) * 8)) = ra[i];
        }
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const int r = lrow + RPT * i;
            *(uint4*)(Bs + r * LDS_LD + ((lchunk ^ swz<BK>(r)) * 8)) = rb[i];
        }
    };

    f32x16_t acc[WMT][WNT];
#pragma unroll
    for (int i = 0; i < WMT; ++i)
#pragma unroll
        for (int jj = 0; jj < WNT; ++jj)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][jj][v] = 0.f;

    // operand rows of this lane: row (32 t + l32) of the wave's A / B block; with 128-byte rows the
    // swizzle key of row + 32 t is the key of the row ^ (4 t & 7), with 64-byte rows it does not change
    const bf16_t* as = As + (wm * WMT * 32 + l32) * LDS_LD;
    const bf16_t* bs = Bs + (wn * WNT * 32 + l32) * LDS_LD;
    const int fa = swz<BK>(wm * WMT * 32 + l32), fb = swz<BK>(wn * WNT * 32 + l32);
    constexpr int TK = BK == 64 ? 4 : 0;   // 256-byte rows: the key is the row's low four bits, the same 32 rows on

    const int kchunks = (k_in + BK - 1) / BK;
    const int nk = KH * KW * kchunks;
    int tap = 0, kc = share * BK;
    if constexpr (KS > 1)
        while (kc >= kchunks * BK) {
            kc -= kchunks * BK;
            ++tap;
        }
    set_tap(tap);
    load_global(tap, kc, share < nk);

    // The first operand slab is requested before anything else: loads return in order, so whatever is issued
    // ahead of it would have to arrive before the slab can go to LDS.
    // epilogue constants, loaded now so their latency hides behind the main loop
    constexpr int COLS = TL::COLS, ST_LD = TL::ST_LD;
    // scale and shift of the tile's columns wait in LDS, not in registers, until the epilogue (registers set the residency)
    if (threadIdx.x < BN) {
        const int n = n0 + tid;
        float vs = 1.f, vh = 0.f;
        if (n < k_out) {
            const long long ti = (long long)lanes.row(g) * tab_ld + (long long)seg * tab_seg + n;
            if (scale) vs = scale[ti];
            if (shift) vh = shift[ti];
        }
        scl[tid] = vs;
        scl[BN + tid] = vh;
    }

    // The residual pieces this lane will add are fetched ahead of the main loop, so that their latency hides behind it
    // instead of sitting between the last matrix instruction and the stores -- except with the 64-deep slabs, where
    // their 16 registers would cost a resident workgroup: there they are requested right after the loop.
    // One share: 8 channels of rows (lane / 8) + 8 i of the wavefront's 32; several: 4 channels of every 16 KS-th row of the tile, few
    // enough to ask for them early.
    constexpr bool RES_EARLY = BK == 32 || KS > 1;
    constexpr int NE = KS == 1 ? 4 : BM / (16 * KS);
    const int srow = lane >> 3, ncol8 = n0 + wn * COLS + (lane & 7) * 8;
    const int ncol4 = n0 + (threadIdx.x & 15) * 4;           // (several shares: one column tile)
    static_assert(COLS == 64, "eight 16-byte pieces a row of the stage");
    static_assert(!F32 || (KS == 1 && !CONV), "fp32 results of linear layers, one share");
    using Piece = typename std::conditional<KS == 1, uint4, uint2>::type;
    Piece rres[HASR ? NE : 1];
    auto fetch_residual = [&](int tm) {
#pragma unroll
        for (int i = 0; i < NE; ++i) {
            const int r = KS == 1 ? wm * WMT * 32 + tm * 32 + srow + 8 * i : ((int)threadIdx.x >> 4) + i * 16 * KS;
            Piece t = {};
            if constexpr (F32) {                             // channels 4 (lane % 8) .. + 3 of either half of the columns
                const int n = n0 + wn * COLS + (lane & 7) * 4;
                if (rowC[r] >= 0) {
                    if (n < k_out) *(uint2*)&t.x = *(const uint2*)(R + rowR[r] + n);
                    if (n + 32 < k_out) *(uint2*)&t.z = *(const uint2*)(R + rowR[r] + n + 32);
                }
            } else {
                const int n = KS == 1 ? ncol8 : ncol4;
                if (n < k_out && rowC[r] >= 0) t = *(const Piece*)(R + rowR[r] + n);
            }
            rres[i] = t;
        }
    };
    // (asked for ahead of the loop's first barrier: the rows of the table are the wavefront's own, or all wavefronts')
    if constexpr (HASR && RES_EARLY) {
        if constexpr (KS > 1 || WCOLS > 1) __syncthreads();
        else wave_sync();
        fetch_residual(0);
    }

    store_lds();
    __syncthreads();
    const int turns = KS > 1 ? (nk + KS - 1) / KS : nk;      // every share as many; a slab past the last is zeros
    for (int kt = 0; kt < turns; ++kt) {
        const bool more = kt + 1 < turns;
        if constexpr (KS == 1) {
            kc += BK;
            if (kc >= k_in) {
                kc = 0;
                ++tap;
                if (more) set_tap(tap);
            }
        } else {
            kc += KS * BK;
            bool next = false;
            while (kc >= kchunks * BK) {
                kc -= kchunks * BK;
                ++tap;
                next = true;
            }
            if (more && next) set_tap(tap);
        }
        if (more) load_global(tap, kc, KS == 1 || share + (kt + 1) * KS < nk);
#pragma unroll
        for (int kk = 0; kk < BK / 16; ++kk) {
            bf16x8_t af[WMT], bfr[WNT];
            const int c = kk * 2 + lhi;
#pragma unroll
            for (int t = 0; t < WMT; ++t) af[t] = *(const bf16x8_t*)(as + t * 32 * LDS_LD + ((c ^ fa ^ ((TK * t) & 7)) * 8));
#pragma unroll
            for (int t = 0; t < WNT; ++t) bfr[t] = *(const bf16x8_t*)(bs + t * 32 * LDS_LD + ((c ^ fb ^ ((TK * t) & 7)) * 8));
#pragma unroll
            for (int i = 0; i < WMT; ++i)
#pragma unroll
                for (int jj = 0; jj < WNT; ++jj)
                    acc[i][jj] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[jj], af[i], acc[i][jj], 0, 0, 0);
        }
        __syncthreads();
        if (more) {
            store_lds();
            __syncthreads();
        }
    }

    // Filters are the instruction's row operand, so a lane holds 4 channels of one row at a time: channels 32 tn + 8 q + 4 lhi of row l32.
    if constexpr (KS > 1) {
        // ---- partial tiles to LDS, added in share order (the loop's last barrier has retired every read of the slabs there)
        float* part = (float*)As;
#pragma unroll
        for (int tn = 0; tn < WNT; ++tn)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *(float4*)(part + (wm * 32 + l32) * TL::PT_LD + tn * 32 + 8 * q + 4 * lhi) =
                    make_float4(acc[0][tn][4 * q], acc[0][tn][4 * q + 1], acc[0][tn][4 * q + 2], acc[0][tn][4 * q + 3]);
        __syncthreads();
        const int cg = threadIdx.x & 15;
        const float4 s4 = *(const float4*)(scl + cg * 4), h4 = *(const float4*)(scl + BN + cg * 4);
        with_act<!CONV>(act, [&](auto actc) {
            constexpr int ACT = decltype(actc)::value;
#pragma unroll
            for (int i = 0; i < NE; ++i) {
                const int r = ((int)threadIdx.x >> 4) + i * 16 * KS;
                const long long coff = rowC[r];
                if (ncol4 >= k_out || coff < 0) continue;
                float4 t = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
                for (int k = 0; k < KS; ++k) {
                    const float4 p = *(const float4*)((const float*)(smem + k * TL::MAIN_BYTES) + r * TL::PT_LD + cg * 4);
                    t.x += p.x; t.y += p.y; t.z += p.z; t.w += p.w;
                }
                float val[4] = {t.x * s4.x + h4.x, t.y * s4.y + h4.y, t.z * s4.z + h4.z, t.w * s4.w + h4.w};
                if constexpr (HASR) add_residual(val, make_uint2(rres[i].x, rres[i].y));
                if (out_f32) {
                    activate<ACT>(val);
                    *(float4*)((float*)C + coff + ncol4) = make_float4(val[0], val[1], val[2], val[3]);
                } else {
                    *(uint2*)((bf16_t*)C + coff + ncol4) = activate_bf16<ACT>(val);
                }
            }
        });
        return;
    }
    // ---- epilogue: a wavefront's 32 x 64 tile through LDS as bf16.  A residual is parked there and every lane adds to its own runs of
    // 4 channels in place; the tile leaves as 16-byte pieces, eight lanes a row.
    // The stage belongs to one wavefront (written and read back by its own lanes, and the main loop's last
    // barrier has already retired every read of the operand tiles it aliases), and a wavefront's LDS accesses
    // complete in order, so only the compiler has to be kept from moving them.
    bf16_t* st = (bf16_t*)smem + wave * 32 * ST_LD;
#pragma unroll
    for (int tm = 0; tm < WMT; ++tm) {
        const int row0 = wm * WMT * 32 + tm * 32;
        if constexpr (HASR) {
            if (!RES_EARLY || tm > 0) fetch_residual(tm);
        }
        if constexpr (F32) {
            // fp32 results go through the stage 32 columns at a time and leave as whole lines, eight lanes a row; a residual is added on the
            // way out.  Stored by the lanes that hold the sums, 16 bytes on each of 32 rows at once -> here, us: 64 images of 197 tokens,
            // 192 -> 768 channels 14.4 -> 11.7, 768 -> 3072 with residual 75.2 -> 68.3; 256 images, 384 -> 1536 100.8 -> 93.4, with residual 136
            // -> 120.  Instances of their own: decided by the argument, this way out spills in the bf16 kernels (the last of these in bf16
            // 88 -> 96).
            constexpr int F_LD = ST_LD / 2;
            float* sf = (float*)st;
            with_act<!CONV>(act, [&](auto actc) {
                constexpr int ACT = decltype(actc)::value;
#pragma unroll
                for (int tn = 0; tn < WNT; ++tn) {
                    const f32x16_t& t = acc[tm][tn];
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int ch = 8 * q + 4 * lhi;
                        const float4 s4 = *(const float4*)(scl + wn * COLS + tn * 32 + ch), h4 = *(const float4*)(scl + BN + wn * COLS + tn * 32 + ch);
                        float val[4] = {t[4 * q] * s4.x + h4.x, t[4 * q + 1] * s4.y + h4.y, t[4 * q + 2] * s4.z + h4.z, t[4 * q + 3] * s4.w + h4.w};
                        if constexpr (!HASR) activate<ACT>(val);
                        *(float4*)(sf + l32 * F_LD + ch) = make_float4(val[0], val[1], val[2], val[3]);
                    }
                    wave_sync();
                    const int n = n0 + wn * COLS + tn * 32 + (lane & 7) * 4;
                    if (n < k_out) {
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            const int row = srow + 8 * i;
                            const long long coff = rowC[row0 + row];
                            float4 v = *(const float4*)(sf + row * F_LD + (lane & 7) * 4);
                            if constexpr (HASR) {
                                float val[4] = {v.x, v.y, v.z, v.w};
                                add_residual(val, tn ? make_uint2(rres[i].z, rres[i].w) : make_uint2(rres[i].x, rres[i].y));
                                activate<ACT>(val);
                                v = make_float4(val[0], val[1], val[2], val[3]);
                            }
                            if (coff >= 0) *(float4*)((float*)C + coff + n) = v;
                        }
                    }
                    wave_sync();
                }
            });
            continue;
        }
        if constexpr (HASR) {
#pragma unroll
            for (int i = 0; i < 4; ++i) *(Piece*)(st + (srow + 8 * i) * ST_LD + (lane & 7) * 8) = rres[i];
            wave_sync();
        }
        with_act<!CONV>(act, [&](auto actc) {
            constexpr int ACT = decltype(actc)::value;
#pragma unroll
            for (int tn = 0; tn < WNT; ++tn)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int ch = tn * 32 + 8 * q + 4 * lhi;
                    const float4 s4 = *(const float4*)(scl + wn * COLS + ch), h4 = *(const float4*)(scl + BN + wn * COLS + ch);
                    const f32x16_t& t = acc[tm][tn];
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
                const long long coff = rowC[row0 + srow + 8 * i];
                if (coff >= 0) *(uint4*)((bf16_t*)C + coff + ncol8) = *(const uint4*)(st + (srow + 8 * i) * ST_LD + (lane & 7) * 8);
            }
        }
        wave_sync();
    }
}

template <int WROWS, int WCOLS, int WMT, int WNT, int BK, int KS, bool CONV, bool HASR, bool F32 = false>
int32_t launch(const GemmArgs& a, int32_t max_mtiles, int32_t max_kout, hipStream_t s) {
    using TL = Tile<WROWS, WCOLS, WMT, WNT, BK, KS>;
    if constexpr (KS == 1 && !CONV && !F32) {
        if (a.out_f32) return launch<WROWS, WCOLS, WMT, WNT, BK, KS, CONV, HASR, true>(a, max_mtiles, max_kout, s);
    }
    auto kern = gemm_kernel<WROWS, WCOLS, WMT, WNT, BK, KS, CONV, HASR, F32>;
    {
        const int32_t rc = ds_reserve_lds((const void*)kern, TL::SMEM, "sliced gemm");
        if (rc) return rc;
    }
    const int ny = a.n_seg * ((max_kout + TL::BN - 1) / TL::BN);
    const unsigned grid = (unsigned)(((max_mtiles + 7) / 8) * ny * 8);
    ProfScope prof(a.K > 1 ? DS_K_GEMM_TAPS : DS_K_GEMM, s);
    hipLaunchKernelGGL(kern, dim3(grid), dim3(NT * KS), TL::SMEM, s, a, ny, max_mtiles);
    DS_CHECK_LAUNCH("sliced gemm");
    return DS_OK;
}

template <int BK, int KS>
int32_t launch_pair(GemmPair& p, const int32_t* kout, hipStream_t s) {
    using TL = Tile<4, 1, 1, 2, BK, KS>;
    auto kern = gemm_kernel<4, 1, 1, 2, BK, KS, true, false, false, GemmPair>;
    {
        const int32_t rc = ds_reserve_lds((const void*)kern, TL::SMEM, "sliced gemm");
        if (rc) return rc;
    }
    unsigned grid[2];
    for (int q = 0; q < 2; ++q) {
        p.ny[q] = (kout[q] + TL::BN - 1) / TL::BN;
        grid[q] = (unsigned)(((p.mtiles[q] + 7) / 8) * p.ny[q] * 8);
    }
    p.split = grid[0];
    ProfScope prof(DS_K_GEMM, s);
    hipLaunchKernelGGL(kern, dim3(grid[0] + grid[1]), dim3(NT * KS), TL::SMEM, s, p, 0, 0);
    DS_CHECK_LAUNCH("sliced gemm");
    return DS_OK;
}

}  // namespace

// The most tiles B samples of `rows` rows can make in T groups: every non-empty group (at most min(B, T)) adds at most
// one partly filled tile to what its rows need.
size_t ds_mtile_capacity(int32_t B, int32_t rows, int32_t T) {
    if (B <= 0 || rows <= 0) return 1;
    const int64_t n = (int64_t)B * rows, g = B < T ? B : T;
    return (size_t)((n - g) / BM + g);
}

namespace {

enum GemmTile { SLAB32, SLAB64, SLAB64_2, SLAB64_4, SLAB128, WIDE32, WIDE64, WIDE64_CONV };

bool is_conv(const GemmArgs& a) { return a.K > 1 || a.stride > 1 || a.pad > 0; }

GemmTile tile_of(const GemmArgs& a, int32_t max_mtiles, int32_t max_kout) {
    const bool conv = is_conv(a);
    // ragged route slices favour the narrow 128x64 tile at high occupancy in every layer of the batch-256 networks.
    // Its slabs are 32 deep for short reductions and 64 deep from 256 reduction steps on: half the barriers and
    // twice the bytes in flight per workgroup outweigh the lower residency there.  Us a pass, 32 deep everywhere -> here: DS-ResNet 33 / 64 /
    // 256 images 811 / 1142 / 2617 -> 737 / 1009 / 2454, DS-ResNet++ 256 images 3002 -> 2848, DS-MBNet++ 96 / 256 images 427 / 797 -> 399 / 753.
    // (a slab never crosses a filter tap: with fewer than 64 channels per tap the deep slab would be mostly padding)
    int kmax = 0;
    for (int t = 0; t < a.gt.T; ++t) kmax = a.gt.k_in[t] > kmax ? a.gt.k_in[t] : kmax;
    const long long taps = (long long)a.K * (a.Kw > 0 ? a.Kw : a.K);
    // (exactly 256 steps: the 64-deep slabs pay only where a residual is streamed as well -- without one the 32-deep kernel keeps six
    // workgroups per compute unit.  64 deep there too / here: DS-ResNet 64 / 96 / 256 images 1012 / 1219 / 2443 and 1008 / 1214 / 2421, DS-ResNet++
    // 64 / 256 images 1107 / 2819 and 1102 / 2802.  From 512 steps on in place of 320 no pass differs)
    const bool deep = kmax >= 64 && (kmax * taps >= 320 || (kmax * taps >= 256 && a.R != nullptr));
    // 128 columns a workgroup, two wavefronts of 64 x 64 either way, so that rows go through LDS half as often, where a launch still has
    // several generations of such workgroups and few of them are half empty.
    // - layers of at most 256 channels whose columns are all in one such tile: 256 images of DS-ResNet 2440 -> 2423 us a pass; with the line at 768
    //   tiles 64 / 96 images (1569 and 2353 row tiles) 1009 / 1213 -> 1015 / 1224, so it stands at 3000
    // - strided KxK layers: 256 images of DS-ResNet 2443 -> 2423, of DS-ResNet++ 2826 -> 2805; with the line at 250 tiles (stage 4's) 128 / 256 images of
    //   DS-ResNet 1469 / 2423 -> 1491 / 2441
    // With a residual, or more columns at stride 1, they lost (stage 3, last 1x1 39.5 -> 49.7 us a launch, stage 4, first 1x1 28.4 -> 37.5,
    // measured before tiles left as 16-byte pieces).
    const long long tiles128 = (long long)max_mtiles * a.n_seg * ((max_kout + 127) / 128) * (a.crowd > 1 ? a.crowd : 1);
    if (!a.R && max_kout > 64) {
        if (!conv && !deep && kmax > 128 && max_kout <= 128 && tiles128 >= 3000) return WIDE32;
        // - linear layers of 768 channels and more, us a call with its bucketing done: 64 / 128 / 256 images of 197 tokens, 768 -> 3072 (2376 tiles and
        //   more) 58.1 / 109.9 / 220.6 -> 52.1 / 95.4 / 192.4; with GELU 63.1 / 120.0 / 242.5 -> 60.5 / 111.3 / 221.8.  From 1000 tiles on they gain as well
        //   (40 images 39.1 -> 35.1, with GELU no change), but there a stage of sixteen route groups lost (DS-ResNet stage 4, first
        //   1x1 of the strided block, 256 images, 1568 tiles, 41.8 -> 50.5).  384 channels: 64 / 128 / 256 images 20.8 / 35.1 / 64.0 -> 21.9 / 34.6 / 62.4, with
        //   GELU 25.8 / 42.2 / 78.0 -> 28.3 / 44.9 / 82.2.
        if (!conv && kmax >= 768 && tiles128 >= 2048) return WIDE64;
        if (taps > 1 && deep && tiles128 >= 768) return WIDE64_CONV;
    }
    if (!deep) return SLAB32;   // 64-wide tile, 32-deep slabs
    // launches of about one generation with long reductions (below): 128-deep slabs halve the number of dependent rounds.  Us a pass, without
    // them / here / without the bound of six workgroups a compute unit: DS-ResNet 96 / 128 / 256 images 1226 / 1479 / 2438, 1214 / 1469 / 2421 and
    // 1225 / 1485 / 2459 (33 / 64 images 732 / 1006, 736 / 1008, 735 / 1012), DS-ResNet++ 256 images 2789 / 2802 / 2854, DS-MBNet++ 256 images 741 / 740 / 783
    const long long wgs = (long long)max_mtiles * a.n_seg * ((max_kout + 63) / 64), slabs = taps * ((kmax + 63) / 64);
    const long long all = wgs * (a.crowd > 1 ? a.crowd : 1);
    // Fewer workgroups than run at once: the slabs of a tile dealt to shares of four wavefronts (not where sums keep one order).
    // A workgroup of four shares has a compute unit to itself, so beyond 256 of them there are two generations: worth it only where a share
    // of half the slabs is a long chain, from 32 slabs on.  Us a pass, one share everywhere / four shares up to 256 workgroups whatever the
    // slabs / here / up to 512 whatever the slabs: DS-ResNet 33 images 760 / 738 / 737 / 752, 64 images 1031 / 1017 / 1009 / 1017, 96 images 1233 /
    // 1230 / 1218 / 1217; DS-ResNet++ 33 images 802 / 793 / 793 / 814, 64 images 1110 / 1102 / 1108 / 1131; DS-MBNet++ 40 images 301 / 301 / 301 / 312.
    // Half and twice all these lines: DS-ResNet 8 / 16 / 33 / 64 / 96 images 533 / 587 / 752 / 1030 / 1231 and 528 / 601 / 760 / 1030 / 1227 (here 526 /
    // 602 / 736 / 1009 / 1214), DS-ResNet++ 33 images 791 and 853 (793), DS-MBNet++ 40 images 301 and 324 (301).
    if (!a.ordered && slabs >= 8 && all <= (slabs >= 32 ? 512 : 256)) return SLAB64_4;
    if (!a.ordered && slabs >= 4 && all <= 512) return SLAB64_2;
    if (kmax >= 512 && wgs <= 256 * 6) return SLAB128;
    return SLAB64;
}

}  // namespace

int32_t ds_launch_gemm(const GemmArgs& a, int32_t max_mtiles, int32_t max_kout, hipStream_t s) {
    if (max_mtiles <= 0 || max_kout <= 0) return DS_OK;
    int kmax = 0;
    for (int t = 0; t < a.gt.T; ++t) kmax = a.gt.k_in[t] > kmax ? a.gt.k_in[t] : kmax;
    const long long taps = (long long)a.K * (a.Kw > 0 ? a.Kw : a.K);
    // 32-bit byte offsets inside the kernel: activations and weights must each span less than 2 GiB
    const long long slots = (long long)max_mtiles * BM / (a.rows > 0 ? a.rows : 1) + 1;
    if (slots * a.a_sample_stride * 2 >= 0x7fffffffLL)
        DS_FAIL(DS_EUNSUPPORTED, "sliced gemm: activation tensor spans 2 GiB or more");
    if (((long long)a.n_seg * a.w_seg_stride + (long long)max_kout * a.w_ld + taps * a.w_tap_stride + kmax) * 2 >= 0x7fffffffLL)
        DS_FAIL(DS_EUNSUPPORTED, "sliced gemm: weight tensor spans 2 GiB or more");
    const bool conv = is_conv(a);
    {
        const int32_t rc = ds_launch_gemm_small(a, max_mtiles, max_kout, s);
        if (rc != DS_EUNSUPPORTED) return rc;
    }
    if (conv) {
        if (!conv_result(a)) DS_FAIL(DS_EUNSUPPORTED, "sliced gemm: convolutions give bf16, without GELU");
        const int32_t rc = ds_launch_conv3(a, max_mtiles, max_kout, s);
        if (rc != DS_EUNSUPPORTED) return rc;
    }
#define DS_GEMM_DISPATCH(...)                                                                          \
    (conv ? (a.R ? launch<__VA_ARGS__, true, true>(a, max_mtiles, max_kout, s)                         \
                 : launch<__VA_ARGS__, true, false>(a, max_mtiles, max_kout, s))                       \
          : (a.R ? launch<__VA_ARGS__, false, true>(a, max_mtiles, max_kout, s)                        \
                 : launch<__VA_ARGS__, false, false>(a, max_mtiles, max_kout, s)))
    switch (tile_of(a, max_mtiles, max_kout)) {
        case WIDE32: return launch<2, 2, 2, 2, 32, 1, false, false>(a, max_mtiles, max_kout, s);
        case WIDE64: return launch<2, 2, 2, 2, 64, 1, false, false>(a, max_mtiles, max_kout, s);
        case WIDE64_CONV: return launch<2, 2, 2, 2, 64, 1, true, false>(a, max_mtiles, max_kout, s);
        case SLAB32: return DS_GEMM_DISPATCH(4, 1, 1, 2, 32, 1);   // 64-wide tile, 32-deep slabs
        case SLAB64_4: return DS_GEMM_DISPATCH(4, 1, 1, 2, 64, 4);
        case SLAB64_2: return DS_GEMM_DISPATCH(4, 1, 1, 2, 64, 2);
        case SLAB128: return DS_GEMM_DISPATCH(4, 1, 1, 2, 128, 1);
        default: return DS_GEMM_DISPATCH(4, 1, 1, 2, 64, 1);
    }
#undef DS_GEMM_DISPATCH
}

int32_t ds_launch_gemm_pair(const GemmArgs& a, int32_t mtiles_a, int32_t kout_a, const GemmArgs& b, int32_t mtiles_b, int32_t kout_b, hipStream_t s) {
    if (mtiles_a <= 0 || mtiles_b <= 0 || kout_a <= 0 || kout_b <= 0 || a.B <= 0 || b.B <= 0) return DS_EUNSUPPORTED;
    const GemmArgs* ps[2] = {&a, &b};
    const int32_t mt[2] = {mtiles_a, mtiles_b}, ko[2] = {kout_a, kout_b};
    for (int q = 0; q < 2; ++q) {
        const GemmArgs& p = *ps[q];
        if (p.K != 1 || p.Kw > 1 || p.pad || p.R || p.ordered || p.n_seg != 1 || !conv_result(p)) return DS_EUNSUPPORTED;
        int kmax = 0;
        for (int t = 0; t < p.gt.T; ++t) kmax = p.gt.k_in[t] > kmax ? p.gt.k_in[t] : kmax;
        // (shorter ones are thin_kernel's; spans as in ds_launch_gemm)
        const long long slots = (long long)mt[q] * BM / (p.rows > 0 ? p.rows : 1) + 1;
        if (kmax <= 128 || slots * p.a_sample_stride * 2 >= 0x7fffffffLL || ((long long)ko[q] * p.w_ld + kmax) * 2 >= 0x7fffffffLL ||
            ds_gemm_small_takes(p, mt[q], ko[q]))
            return DS_EUNSUPPORTED;
    }
    // the tile that either layer takes alone, so that pairing changes no sum
    const GemmTile tile = tile_of(a, mtiles_a, kout_a);
    if (tile != tile_of(b, mtiles_b, kout_b)) return DS_EUNSUPPORTED;
    GemmPair p;
    for (int q = 0; q < 2; ++q) { p.p[q] = *ps[q]; p.mtiles[q] = mt[q]; }
    switch (tile) {
        case SLAB32: return launch_pair<32, 1>(p, ko, s);
        case SLAB64: return launch_pair<64, 1>(p, ko, s);
        case SLAB128: return launch_pair<128, 1>(p, ko, s);
        case SLAB64_2: return launch_pair<64, 2>(p, ko, s);
        default: return DS_EUNSUPPORTED;
    }
}
