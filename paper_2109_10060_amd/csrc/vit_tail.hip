// The rest of a transformer block behind its attention, in one kernel (Section 3.2, Eq. 15-19):
//   x += proj(o);  x += fc2(gelu(fc1(LN2(x))));  and where it pays the next block's Q/K/V of LN1(x)
// for every route group, slices as everywhere: the leading block of the stored weights.
//
// As four launches (projection, LayerNorm, two linear layers) a block moved the residual stream five times and the hidden
// activations twice through memory, and its reductions of 192..416 channels spent their time in the head and the epilogue
// of the workgroups.  Here a workgroup owns BM = 32 R rows from the attention output to the block's own; the hidden layer
// never leaves the compute unit (HC columns at a time in LDS).
//
// What bounds it: the weights' way from L2 into a compute unit (about 50 bytes a clock, all of the block's weights once per
// workgroup), the matrix pipes and the vector ALU (GELU, LayerNorm), in that order and only partly side by side.  So the
// weights are kept in operand order (32 rows x 16 channels = 64 lanes x 16 bytes, tiles of 1 KiB): a wavefront reads each
// operand as one contiguous kilobyte straight into registers, D of them in flight, and LDS serves the activations alone.
// Each of the NW = 12 (13 above 384 channels) wavefronts owns one 32-column block of the block's width and of every
// HC = 32 NW columns of the hidden layer; R row blocks share every weight operand.
// Around the products a workgroup has nothing beside it on its compute unit, so what it waits for is kept off its path: the
// residual rows wait in a hidden tile, which is free until the MLP, LayerNorm weights in LDS, biases in a register a lane.
//
// The products of a wavefront are one stream of operands: the last turn of each asks for the first operands of the next, across
// LayerNorm, GELU and barriers.  Behind the block a workgroup still has its rows: it normalises them for the next block and multiplies
// them with that block's Q/K/V weights, stored from registers as vit_linear_kernel stores them.
// A workgroup of 384 channels and 1536 hidden ones lives 122 thousand clocks: rows 9, projection 8, LayerNorm 5, MLP 65, rows out and
// LayerNorm 7, Q/K/V 22; the matrix pipe is busy for 55 of them, the vector ALU for about 45.  A loop of these loads, LDS reads and products
// alone takes 57 bytes a clock from L2 and keeps the pipe at 90 %; here the mean is 35 to 45, because a wait for one operand is a wait for
// everything asked for before it.  What that took: LDS reads issued a step ahead (the compiler sank them behind the products), no branch
// that gives out the operands under way (they were moved there, and a move waits for them), requests for rows and constants and stores
// without branches, six operands in flight for four, two hidden tiles and so one barrier a tile for two.  us a pass, before -> now: 256
// images of DS-ViT 2322 -> 2217, on another card 2444 -> 2322; 60 to 100 images 1074 -> 975; 256 images of DS-ViT++ (13 wavefronts: one
// hidden tile, four in flight; of its 128 registers a lane 16 leave for scratch ahead of the hidden columns and come back behind them, once a
// workgroup) 3522 -> 3440.  Eight operands in flight 2350 for 2322 at 256 images.  Q/K/V blocks dealt out as wavefronts
// come free instead of in turn: no change.
//
// Sums run in the order of gemm_kernel's and layernorm16_kernel's, so the results are the same bits.
#include "tile_out.h"
#include "vit_rows.h"

namespace {

typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

// Pitches of the activation tile and of the hidden tiles: two of them, or one where 13 wavefronts leave no LDS for a second (two of 12 column
// blocks are five rounds for 1664 hidden channels where one of 13 is four: 256 images of DS-ViT++ 3512 us a pass, 3616 with two); 8
// elements behind the last one for the read-ahead of its last row.
template <int NW, int R, int D, int KR>
struct TailTile {
    static constexpr bool TWO = NW <= 12;
    static constexpr int KA = KR;                           // channels of a row
    static constexpr int PA = tile_pitch(KA, D), PH = tile_pitch(32 * NW, D);
    static constexpr int NORM = 32 * R * (PA + (TWO ? 2 : 1) * PH) + 8; // LayerNorm weights: gamma, then beta
    static constexpr int BIAS = NORM + 2 * 2 * KA;          // of each wavefront's columns
    static constexpr int SMEM = BIAS * 2 + NW * 32 * 4;
    static_assert(SMEM <= 160 * 1024, "LDS of a compute unit");
};

// k channels of weights of a 32-column block
struct Stream {
    const bf16_t* w;
    int k;
};

// NW wavefronts (one column block of 32 each), 32 R rows, D operands of a wavefront in flight, rows of up to KR channels
template <int NW, int R, int D, int KR>
__global__ __launch_bounds__(64 * NW, (NW + 3) / 4) void vit_tail_kernel(const VitTailArgs a) {
    using Tile = TailTile<NW, R, D, KR>;
    constexpr int BM = 32 * R, HC = 32 * NW, PA = Tile::PA, PH = Tile::PH, KA = Tile::KA, RP = 4 * NW, NI = (BM + RP - 1) / RP;   // RP: rows of a row phase
    extern __shared__ __attribute__((aligned(16))) char smem[];
    bf16_t* As = (bf16_t*)smem;                         // [BM][PA]
    constexpr bool TWO = Tile::TWO;
    bf16_t* Hs = As + BM * PA;                          // [TWO ? 2 : 1][BM][PH]
    float* gs = (float*)(As + Tile::NORM);              // [2][KA]

    const int4 me = ds_tile_record_of(a.offsets, a.gt.T, a.rows, (int)blockIdx.x, BM);
    if (me.x < 0) return;
    const int g = me.x, grow0 = me.y, slot0 = me.z, rows_g = me.w;
    const int kin = a.gt.k_in[g], de = a.gt.k_out[g], hid = a.gt.row[g];
    if (de <= 0) return;

    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, l32 = lane & 31, lhi = lane >> 5;
    const int l16 = tid & 15, prow = tid >> 4;          // row phases: 16 lanes a row, RP rows at a time
    const bool con = w * 32 < de;                        // this wavefront has a column block


    // ---- rows of this thread's 16-lane group: attention output and residual rows to the two tiles ---------------------------
    // Rows, constants and outputs go through descriptors of the tile's first sample: what lies outside a slice or a group is an offset out
    // of range.  Without a branch around them the requests travel together, and the number in flight is known wherever one is waited
    // for -- behind a branch every wait for the weights' ring would be one for the rows and stores as well.
    constexpr uint32_t OOB = 0x80000000u;
    const int first = ds_quotient(grow0, a.rows);                    // (of the group; rows of a tile count from there)
    auto window = [](const void* p, int64_t elements) {
        return __builtin_amdgcn_make_buffer_rsrc((void*)((const bf16_t*)p + elements), 0, 0x7fffffff, 0x00020000);
    };
    const __amdgpu_buffer_rsrc_t rx = window(a.x, (int64_t)(slot0 + first) * a.x_ss);
    uint32_t xoff[NI];                                   // of this lane's first 8 channels; out of range: no such row
    // rows of x, the residual of both sums, in a tile of LDS
    auto x_rows = [&](uint4 (&q)[NI][4]) {
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int k = 0; k < 4; ++k)
                q[i][k] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rx, (int)((k * 16 + l16) * 8 < de ? xoff[i] + k * 256 : OOB), 0, 0));
    };
    auto to_tile = [&](const uint4 (&q)[NI][4], bf16_t* tile, int pitch, int width) {
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int ch = (k * 16 + l16) * 8;
                if (ch < width && (BM % RP == 0 || prow + RP * i < BM)) *(uint4*)(tile + (prow + RP * i) * pitch + ch) = q[i][k];
            }
    };
    {
        uint4 q[NI][4], xr[NI][4];
        const __amdgpu_buffer_rsrc_t ro = window(a.o, (int64_t)(slot0 + first) * a.o_ss);
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const bool in = BM % RP == 0 || prow + RP * i < BM;
            const int m = grow0 + prow + RP * i, sl = ds_quotient(m, a.rows), p = m - sl * a.rows;
            const bool live = in && m < rows_g;
            xoff[i] = live ? (uint32_t)(((sl - first) * a.x_ss + (int64_t)p * de + l16 * 8) * 2) : OOB;
            const uint32_t ooff = live ? (uint32_t)(((sl - first) * a.o_ss + (int64_t)p * a.o_ld + l16 * 8) * 2) : OOB;
#pragma unroll
            for (int k = 0; k < 4; ++k)
                q[i][k] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(ro, (int)((k * 16 + l16) * 8 < kin ? ooff + k * 256 : OOB), 0, 0));
        }
        x_rows(xr);
        for (int i = tid; i < de; i += 64 * NW) {
            gs[i] = a.g2[i];
            gs[KA + i] = a.be2[i];
        }
        to_tile(q, As, PA, PA);                          // zeros beyond the slice
        to_tile(xr, Hs, PH, de);
    }
    auto x_out = [&](int i, int k, const uint4& q) {     // 8 channels of a row that this thread fetched
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, q), rx, (int)((k * 16 + l16) * 8 < de ? xoff[i] + k * 256 : OOB), 0, 0);
    };

    // ---- acc2[r] += W[column block w] . act^T over K channels, 16 a step -----------------------------------------------------
    f32x16_t acc2[R];
    auto clear2 = [&]() {
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc2[r][v] = 0.f;
    };
    // Every step is straight-line code: operand requests are unconditional (a step past the end asks for an address out of
    // range and gets zeros without traffic), so the number in flight is known where a product waits for the oldest, and the
    // LDS reads of a step are issued ahead of the products of the step before it.  The number of steps is rounded up to D; the
    // extra steps multiply zero weights with the zeros behind the slice (tile_pitch).
    const uint32_t lane16 = (uint32_t)lane * 16;
    // A product's last turn asks for the first operands of the one behind it, so a ring is started once.
    bf16x8_t ring[D];
    auto start = [&](const Stream& t) {
        const __amdgpu_buffer_rsrc_t rs = weight_row(t.w, 0, t.k);
#pragma unroll
        for (int j = 0; j < D; ++j) ring[j] = weight_tile(rs, lane16 + j * 1024);
    };
    auto walk = [&](f32x16_t (&acc)[R], const Stream& t, const Stream& next, const bf16_t* act, int pitch) __attribute__((always_inline)) {
        const bf16_t* base = act + l32 * pitch + lhi * 8;
        bf16x8_t f[2][R];
#pragma unroll
        for (int r = 0; r < R; ++r) f[0][r] = *(const bf16x8_t*)(base + r * 32 * pitch);
        int k0 = 0;
        bool more;
        do {                                             // (no channels: one turn of zero weights, its sums are not used)
            more = k0 + 16 * D < t.k;
            const __amdgpu_buffer_rsrc_t rs = weight_row(more ? t.w : next.w, 0, more ? t.k : next.k);
            const uint32_t off = lane16 + (more ? k0 * 64 + D * 1024 : 0);
#pragma unroll
            for (int j = 0; j < D; ++j) {
#pragma unroll
                for (int r = 0; r < R; ++r) f[(j + 1) & 1][r] = *(const bf16x8_t*)(base + r * 32 * pitch + k0 + (j + 1) * 16);
                __builtin_amdgcn_sched_barrier(0);       // (the compiler would sink the reads to their use)
#pragma unroll
                for (int r = 0; r < R; ++r) acc[r] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[j], f[j & 1][r], acc[r], 0, 0, 0);
                ring[j] = weight_tile(rs, off + j * 1024);
                __builtin_amdgcn_sched_barrier(0);
            }
            k0 += 16 * D;
        } while (more);
    };
    // Biases of a wavefront's 32 columns travel beside a product in one register a lane and reach the lanes that add them, 4 channels at a
    // time, through the wavefront's own line of LDS.
    float* line = (float*)(As + Tile::BIAS) + w * 32;
    auto columns = [&](const float* v, int c0, int n) {
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)v, 0, n * 4, 0x00020000);
        return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, (c0 + l32) * 4, 0, 0));
    };
    auto bias_of = [&](int q) { return *(const float4*)(line + 8 * q + 4 * lhi); };
    auto to_line = [&](float v) {
        wave_sync();                                     // (what was there has been read)
        line[l32] = v;
        wave_sync();
    };
    // tile (in LDS, bf16) = tile + acc2 + bias on the elements this lane accumulated
    auto add_columns = [&](float cst, bf16_t* tile, int pitch) {
        if (!con) return;
        to_line(cst);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int ch = w * 32 + 8 * q + 4 * lhi;
            if (ch >= de) continue;
            const float4 h = bias_of(q);
#pragma unroll
            for (int r = 0; r < R; ++r) {
                uint2* p = (uint2*)(tile + (r * 32 + l32) * pitch + ch);
                const uint2 res = *p;
                const f32x16_t& t = acc2[r];
                float v0 = t[4 * q] + h.x, v1 = t[4 * q + 1] + h.y, v2 = t[4 * q + 2] + h.z, v3 = t[4 * q + 3] + h.w;
                v0 += __uint_as_float(res.x << 16);
                v1 += __uint_as_float(res.x & 0xffff0000u);
                v2 += __uint_as_float(res.y << 16);
                v3 += __uint_as_float(res.y & 0xffff0000u);
                *p = make_uint2(f2bf2(v0, v1), f2bf2(v2, v3));
            }
        }
    };

    // ---- projection + residual ------------------------------------------------------------------------------------------
    // the columns behind the hidden tile's own, which the extra steps of a full width multiply
    constexpr int PADS = (PH - 8 - HC) / 8;
    if constexpr (PADS > 0)
        for (int i = tid; i < BM * PADS; i += 64 * NW) *(uint4*)(Hs + i / PADS * PH + HC + i % PADS * 8) = make_uint4(0, 0, 0, 0);
    clear2();
    // (no channels: no traffic)
    auto stream = [](const bf16_t* w, int t0, int k) { return Stream{w + (int64_t)t0 * 512, k}; };
    // (held: read again from the arguments they cost a round trip to the scalar cache at every product)
    const bf16_t *w1 = a.w1 + (int64_t)(w * a.kb1) * 512, *w2 = a.w2 + (int64_t)(w * a.kb2) * 512;
    const float *b1 = a.b1, *b2 = a.b2;
    int step1 = NW * a.kb1;
    ds_hold(w1, w2, b1, b2, step1);
    const Stream first_fc1 = stream(w1, 0, w * 32 < hid ? de : 0);
    const Stream sp = stream(a.wp, w * a.kbp, con ? kin : 0);
    start(con ? sp : first_fc1);
    float cst = columns(a.bp, w * 32, de);
    __syncthreads();
    if (con) walk(acc2, sp, first_fc1, As, PA);
    add_columns(cst, Hs, PH);                            // x waits in the hidden tile
    __syncthreads();
    // ---- x to memory, LN2 in place ---------------------------------------------------------------------------------------
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        if (BM % RP != 0 && prow + RP * i >= BM) continue;     // whole 16-lane groups
        float v[4][8];
        uint4 o[4];
        const bf16_t* sum = Hs + (prow + RP * i) * PH;
        bf16_t* row = As + (prow + RP * i) * PA;
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int ch = (k * 16 + l16) * 8;
            if (ch < de) {
                const uint4 q = *(const uint4*)(sum + ch);
                x_out(i, k, q);
                unpack8(q, v[k]);
            }
        }
        row_norm(v, de, l16, a.eps, gs, gs + KA, o);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int ch = (k * 16 + l16) * 8;
            if (ch < de) *(uint4*)(row + ch) = o[k];
            else if (ch < PA) *(uint4*)(row + ch) = make_uint4(0, 0, 0, 0);
        }
    }
    __syncthreads();

    // ---- MLP, HC hidden columns at a time ----------------------------------------------------------------------------------
    // With two hidden tiles there is one barrier a tile: a wavefront that is through with fc2 of one makes its block of the next, its GELU
    // beside the others' products.  Of a SIMD's three wavefronts the second makes its block first (late): 60 to 100 images of DS-ViT 985 -> 975
    // us a pass, 256 images 2281 -> 2276.
    clear2();
    const int nchunk = (hid + HC - 1) / HC;
    const bool more = (a.next >> g) & 1;
    // the next block's Q/K/V: three segments of nb column blocks, NW blocks at a time
    const int nb = (kin + 31) / 32;
    auto qkv = [&](int p) { return stream(a.wq, (p / nb * a.segq + p % nb) * a.kbq, more && p < 3 * nb ? de : 0); };
    // (Every wavefront multiplies at every turn, whether it has columns or not, and nothing else stands around the products: where the
    // operands under way come out of a branch they are moved, and a move waits for them.)
    auto fc1 = [&](int hc) { return stream(w1, hc * step1, hid - hc * HC > w * 32 ? de : 0); };
    auto fc2 = [&](int hc) { return stream(w2, hc * 2 * NW, con ? min(HC, hid - hc * HC) : 0); };
    const bool late = TWO && w >> 2 == 1;
    auto residual = [&]() {
        // the residual rows of the last sum (this thread wrote them itself after the projection): every wavefront is past its
        // last read of the activation tile
        uint4 xr[NI][4];
        x_rows(xr);
        to_tile(xr, As, PA, de);
        __builtin_amdgcn_s_waitcnt(0x0f70);              // vmcnt(0), here and not behind the branch, where it would be one for the operands under way
    };
    // The barrier of a turn.  The hardware counts arrivals, wherever in the code they are: a late wavefront comes to it behind its fc2, the
    // others ahead of theirs, and every wavefront comes once a turn.  (Inside one wavefront the place is the same for all lanes.)
    auto turn = [&]() {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
    };
    Stream cur = fc1(0);
    for (int hc = 0; hc < nchunk; ++hc) {
        const bool last = hc + 1 == nchunk;
        const int hb = hc * NW + w;                      // 32-column block of the hidden layer
        const int two = late ? hc - 1 : hc;              // whose fc2
        const Stream ahead = last ? (late ? fc2(hc) : qkv(w)) : fc1(hc + 1), s2 = two < 0 ? ahead : fc2(two);
        bf16_t* tile = Hs + (TWO ? hc & 1 : 0) * (BM * PH);
        f32x16_t acc1[R];
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc1[r][v] = 0.f;
        cst = columns(b1, hb * 32, hid);
        walk(acc1, cur, s2, As, PA);
        cur = ahead;
        if (!TWO && hc > 0) __syncthreads();             // the previous columns have been read
        to_line(cst);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int ch = hb * 32 + 8 * q + 4 * lhi;
            const float4 h = bias_of(q);
#pragma unroll
            for (int r = 0; r < R; ++r) {
                uint2 o = make_uint2(0, 0);
                if (ch < hid)
                    o = gelu_bf16x4(acc1[r][4 * q] + h.x, acc1[r][4 * q + 1] + h.y, acc1[r][4 * q + 2] + h.z, acc1[r][4 * q + 3] + h.w);
                *(uint2*)(tile + (r * 32 + l32) * PH + w * 32 + 8 * q + 4 * lhi) = o;
            }
        }
        if (!late) {
            turn();
            if (last) residual();
        }
        if (two >= 0) walk(acc2, s2, ahead, Hs + (TWO ? two & 1 : 0) * (BM * PH), PH);
        if (late) turn();
    }
    if (late) {
        residual();
        walk(acc2, cur, qkv(w), Hs + ((nchunk - 1) & 1) * (BM * PH), PH);
    }
    cst = columns(b2, w * 32, de);
    __syncthreads();
    add_columns(cst, As, PA);
    if (more)
        for (int i = tid; i < de; i += 64 * NW) {
            gs[i] = a.g1[i];
            gs[KA + i] = a.be1[i];
        }
    __syncthreads();
    // ---- x to memory, the next block's LN1 in place -------------------------------------------------------------------------
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        if (BM % RP != 0 && prow + RP * i >= BM) continue;     // whole 16-lane groups
        bf16_t* row = As + (prow + RP * i) * PA;
        float v[4][8];
        uint4 o[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int ch = (k * 16 + l16) * 8;
            if (ch < de) {
                const uint4 q = *(const uint4*)(row + ch);
                x_out(i, k, q);
                unpack8(q, v[k]);
            }
        }
        if (!more) continue;
        row_norm(v, de, l16, a.eps, gs, gs + KA, o);
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int ch = (k * 16 + l16) * 8;
            if (ch < de) *(uint4*)(row + ch) = o[k];           // (zeros behind the slice are still there)
        }
    }
    if (!more) return;
    __syncthreads();
    const bf16_t* q0 = a.qkv + (int64_t)(slot0 + first) * a.q_ss;
    uint32_t qoff[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int m = grow0 + r * 32 + l32, sl = ds_quotient(m, a.rows);
        qoff[r] = m < rows_g ? (uint32_t)(((sl - first) * a.q_ss + (int64_t)(m - sl * a.rows) * a.q_ld + 8 * lhi) * 2) : OOB;
    }
    for (int p = w; p < 3 * nb; p += NW) {
        const int seg = p / nb, n0 = (p - seg * nb) * 32;
        clear2();
        cst = columns(a.bq + (int64_t)seg * a.q_ld, n0, kin);
        walk(acc2, qkv(p), qkv(p + NW), As, PA);
        to_line(cst);
        const __amdgpu_buffer_rsrc_t rq = window(q0, (int64_t)seg * a.q_seg + n0);
#pragma unroll
        for (int q = 0; q < 4; q += 2) {
            const bool in = n0 + 8 * q + 8 * lhi < kin;
            const float4 h[2] = {bias_of(q), bias_of(q + 1)};
#pragma unroll
            for (int r = 0; r < R; ++r) {
                uint32_t lo[2], hi[2];
#pragma unroll
                for (int e = 0; e < 2; ++e) {
                    const f32x16_t& t = acc2[r];
                    const int b = 4 * (q + e);
                    lo[e] = f2bf2(t[b] + h[e].x, t[b + 1] + h[e].y);
                    hi[e] = f2bf2(t[b + 2] + h[e].z, t[b + 3] + h[e].w);
                }
                // channels 8 q .. + 7 to the lower half's lane, the next eight to the upper half's
                const auto a0 = __builtin_amdgcn_permlane32_swap(lo[0], lo[1], false, false);
                const auto a1 = __builtin_amdgcn_permlane32_swap(hi[0], hi[1], false, false);
                __builtin_amdgcn_raw_buffer_store_b128(u32x4_t{a0[0], a1[0], a0[1], a1[1]}, rq, (int)(in ? qoff[r] + 16 * q : OOB), 0, 0);
            }
        }
    }
}

template <int NW, int R, int D, int KR>
int32_t launch(const VitTailArgs& a, int64_t tiles, hipStream_t s) {
    constexpr int SMEM = TailTile<NW, R, D, KR>::SMEM;
    const int32_t rc = ds_reserve_lds((const void*)vit_tail_kernel<NW, R, D, KR>, SMEM, "transformer block tail");
    if (rc) return rc;
    ProfScope prof(DS_K_TAIL, s);
    hipLaunchKernelGGL((vit_tail_kernel<NW, R, D, KR>), dim3((unsigned)tiles), dim3(64 * NW), SMEM, s, a);
    DS_CHECK_LAUNCH("transformer block tail");
    return DS_OK;
}

}  // namespace

// The next block's Q/K/V behind the block, or in a launch of its own (vit_linear_kernel), which reads the rows again and takes a
// generation of workgroups more, but spreads over more of them.  So it rides along from about the tiles on at which a launch of its own no longer has
// compute units to spread to; with 13 wavefronts, where 36 column blocks are three rounds of which one is mostly idle, later.  Us a pass of
// DS-ViT, own launch / here: 8 images (57 tiles of 32 rows) 484 / 506, 9 images (64) 561 / 546, 10 images 586 / 538, 16 images 574 / 575, 17 images 668 / 603, 32
// images 772 / 667, 64 images 969 / 879, 256 images 2445 / 2292; DS-ViT++ 15 / 19 images (107, 135) 946 / 970 and 973 / 995, 20 images (142) 1002 / 985, 32
// images 1073 / 1004, 256 images 3717 / 3561; 13 heads of 32 beside 384 channels, 10 / 16 images 652 / 657 and 672 / 671, 18 images 721 / 682.  Parts of a batch
// count together: 32 images in two 731 / 669, 128 in four 1500 / 1286, 256 in four 2420 / 2290, in two 2205 / 2264.
bool ds_vit_tail_qkv(const GroupTable& gt, int32_t B, int32_t rows, int32_t crowd) {
    int dmax = 0;
    for (int t = 0; t < gt.T; ++t) dmax = gt.k_out[t] > dmax ? gt.k_out[t] : dmax;
    const int64_t groups = B < gt.T ? B : gt.T, tiles = ((int64_t)B * rows - groups) / 32 + groups;
    return tiles * (crowd > 1 ? crowd : 1) >= (dmax > 384 ? 140 : 60);
}

// Rows per workgroup.  A workgroup streams all weights of the block whatever its rows (2.7 MB at full width), and when all compute
// units do so at once the L2s give each about 30 bytes a clock, half of what 64 rows could use; so more rows each are better --
// as long as there is a workgroup for nearly every compute unit and the last ones end together.  How many tiles there are, and how long each
// takes, is up to the routes, which the host does not know: the line goes by the most there can be.  Us a pass, 32 / 64 rows, routes spread
// evenly | half of the images on the narrowest | all on the narrowest | all on the widest: DS-ViT 56 images (219 tiles) 815 / 853 | 735 / 855 |
// 574 / 468 | 1298 / 908, 60 images (231) 856 / 854 | 784 / 855 | 574 / 472 | 1303 / 925, 64 images (244) 872 / 864 | 788 / 860 | 577 / 478 | 1308 /
// 943, 71 images (265) 965 / 913 evenly; DS-ViT++ 70 images (223) 1304 / 1389 | 1157 / 1373 | 814 / 717 | 2043 / 1530, 72 images (229) 1271 / 1351 | 1131 /
// 1339 | 782 / 680 | 2004 / 1517, 78 images (247) 1413 / 1455 | 1200 / 1408 | 834 / 738 | 2099 / 1689, 86 images (272) 1649 / 1553 evenly.  On one route,
// 32 rows are more tiles than compute units, all of one length: a second generation that is half empty, 15 to 39 % of a pass here, where 64 rows cost
// up to 19 %.  The line is at 224; at 248 batches on one route took up to a quarter more than they had.  96 rows leave no LDS for the LayerNorm weights: 64 images 1267 us against 1046
// with 64 rows, 192 images 2016 against 2039, 256 images 2587 against 2530 on one card and 2492 against 2485 on another.  (See
// profiles/dispatch_choices.txt.)  Parts of a batch that run side by side fill the compute units together, if not
// evenly.  Us a pass, 32 / 64 rows, two parts and four (tiles of 64 rows in all of them): DS-ViT 64 images (260, 260) 853 / 837 and 907 / 882, 72
// images (292, 292) 924 / 884 and 893 / 887, 80 images (324, 324) 997 / 908 and 1016 / 965, 96 images 1108 / 1025 and 1137 / 1038, 160 images
// 1750 / 1503 in four; DS-ViT++ 64 images in two (212) 1147 / 1308, 80 images (262, 276) 1388 / 1421 and 1467 / 1423, 96 images 1586 / 1555 and 1641 /
// 1582.  (Parts of unequal size each count the others as being of their own: 72 images of DS-ViT++ in two are 40 and 32, which take one each, 1431
// where both with 32 rows take 1272 and both with 64 take 1356.)
int32_t ds_launch_vit_tail(const VitTailArgs& a, int32_t B, hipStream_t s) {
    int dmax = 0, kmax = 0;
    for (int t = 0; t < a.gt.T; ++t) {
        if (a.gt.k_out[t] <= 0) continue;
        dmax = a.gt.k_out[t] > dmax ? a.gt.k_out[t] : dmax;
        kmax = a.gt.k_in[t] > kmax ? a.gt.k_in[t] : kmax;
        if (a.gt.k_in[t] > VIT_K_MAX || a.gt.k_out[t] > VIT_K_MAX || a.gt.row[t] <= 0 || (a.gt.k_in[t] % 16) || (a.gt.k_out[t] % 8) ||
            (a.gt.row[t] % 8))
            return DS_EUNSUPPORTED;
    }
    const int64_t groups = B < a.gt.T ? B : a.gt.T, n = (int64_t)B * a.rows;
    auto tiles = [&](int bm) { return (n - groups) / bm + groups; };
    const bool two = tiles(64) >= 224 || (a.crowd > 1 && tiles(64) * a.crowd >= (dmax > 384 ? 270 : 300));
    // Two workgroups a compute unit from about a generation of them on (512): below, a tile alone on its compute unit takes longer there (384 channels 78
    // us against 67, 192 channels 36 against 30).  How many tiles there are is up to the routes (as many as groups fewer than counted here).
    // us a pass, one workgroup | two: DS-ViT 128 images (441 tiles counted) 1197 | 1248, 144 (490) 1331 | 1344, 160 (540) 1546 | 1450, 176 (589) 1631 |
    // 1625, 216 (712) 1867 | 1867, 256 (836) 2197 | 2081; half of the images on the narrowest route 160 images 1226 | 1268, 192 (638) 1380 | 1383, 256 1773 |
    // 1702; all on the widest 128 images 1752 | 1678, on the narrowest 767 | 715.  DS-ViT++ 144 images (451) 2079 | 2164, 160 (500) 2224 | 2247, 168 (525) 2511 |
    // 2341, 184 (574) 2580 | 2402; half on the narrowest 160 images 1896 | 2131, 192 (599) 2242 | 2247.  Parts of a batch count together: DS-ViT
    // 128 images in two (490) 1228 | 1317, 192 in two (685) 1707 | 1627, in four (780) 1759 | 1657, DS-ViT++ 160 in two (508) 2080 | 2218, 192 in two (606) 2544 | 2410.
    if (tiles(64) * (a.crowd > 1 ? a.crowd : 1) >= 576) return ds_launch_vit_duo(a, tiles(64), dmax > kmax ? dmax : kmax, s);
    if (dmax > 384)                                      // 13 column blocks: 128 registers per lane, at most 64 rows
        return two ? launch<13, 2, 4, VIT_K_MAX>(a, tiles(64), s) : launch<13, 1, 4, VIT_K_MAX>(a, tiles(32), s);
    // attention wider than the output's twelve column blocks: rows of 416 channels leave LDS for four operands' turns beside two hidden tiles.
    // 13 wavefronts -> here, 13 heads of 32 beside an embedding of 384, us a pass: 16 images 719 -> 670, 64 images 1040 -> 1010, 128 images 1688 ->
    // 1532, 256 images 3049 -> 2835
    if (kmax > 384) return two ? launch<12, 2, 4, VIT_K_MAX>(a, tiles(64), s) : launch<12, 1, 8, VIT_K_MAX>(a, tiles(32), s);
    return two ? launch<12, 2, 6, 384>(a, tiles(64), s) : launch<12, 1, 8, 384>(a, tiles(32), s);
}
