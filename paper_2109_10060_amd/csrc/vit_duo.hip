// vit_tail_kernel's work (the rest of a transformer block behind its attention, with the next block's Q/K/V) for launches of two generations
// and more: two workgroups a compute unit, each of four wavefronts and 64 rows, so that one multiplies while the other waits for rows,
// normalises or stores.  Same arguments, same tiles, same bits.
//
// What bounds it: a wavefront issues a vector instruction every 5.4 clocks, whatever the instruction and however its operands come; a second
// wavefront on the SIMD doubles that.  With one twelve-wavefront workgroup a compute unit a tile of 192 channels took 45 % of the time of one of 384
// with six times the products: rows, LayerNorms and stores, with nothing beside them.  Here
//   * a wavefront owns every fourth 32-column block, up to NB of them (2 up to 256 channels, 3 up to 384, 4 up to 416; each in a body of its
//     own): an operand read from LDS serves NB products, and the weights (operand order, straight into registers, D tiles in flight) come at
//     the 64 bytes a clock of the vector cache that 64 rows need at the full matrix rate;
//   * the hidden layer goes by 128 columns (HC), one block a wavefront, through one tile of LDS: 71 KiB a workgroup, 76 above 384 channels;
//   * GELU of the next columns stands between the products of fc2 of the last ones, an instruction stream of a dozen vector instructions a
//     product (walk_tile); by one polynomial without a check (gelu_poly.h) it is 16 instructions a value;
//   * LayerNorms and sums run without branches, two rows side by side.
// Registers are what it is short of (256 a lane): a value that lives through the hidden columns goes to scratch, and to wait for it there is to
// wait for the operands asked for before it.  So rows' addresses are in LDS and each phase works out its lanes' places anew (place()).
//
// Clocks of a workgroup's phases, alone on a compute unit | two beside each other, DS-ViT, 384 channels and 1536 hidden ones: rows 9.0 | 15.7 thousand,
// projection 5.9 | 8.0, residual and LayerNorm 11.1 | 14.1, MLP 89 | 122, residual and LayerNorm 11.5 | 11.5, Q/K/V 31 | 31: 157 | 203, of
// which the matrix pipe is busy for 55 of each.  192 channels and 384 hidden ones: 60 | 74.  A launch of 493 tiles (160 images on one route) of the
// widest route 134 -> 119 us, of the narrowest 60 -> 46.  us a pass at 256 images, vit_tail_kernel -> here: DS-ViT 2197 -> 2081 (half of the images on the
// narrowest route 1773 -> 1702, all on the widest 3722 -> 3326, on the narrowest 1417 -> 1266, two parts 2246 -> 2041), DS-ViT++ 3450 -> 3003.
// Six wavefronts with two blocks each and 168 registers never shared a compute unit: the second workgroup's first wavefronts want the same SIMDs.
#include "tile_out.h"
#include "vit_rows.h"
#include <type_traits>

namespace {

typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

constexpr int NW = 4, HC = 32 * NW;

template <int R, int KR>
struct DuoTile {
    static constexpr int PA = KR + 8, PH = HC + 8;
    static constexpr int NORM = 32 * R * (PA + PH) + 32;    // LayerNorm weights: gamma, then beta
    static constexpr int BIAS = NORM + 2 * 2 * KR;          // of each wavefront's columns
    static constexpr int ROWS = BIAS * 2 + NW * 128 * 4;   // (bytes) where the rows of x are
    static constexpr int SMEM = ROWS + 32 * R * 4;
    static_assert(SMEM <= 80 * 1024, "half of a compute unit's LDS");
    // (reads ahead end up to 16 channels into the row behind, of one block 32: behind the last row of the hidden tile the 32 elements under NORM)
};

// k channels of weights of up to four 32-column blocks
struct Stream {
    const bf16_t* w[4];
    int k, n;        // channels, blocks
};

// NB: column blocks of a wavefront at most, D: operands in flight, KR: channels of a row at most
template <int NB, int D, int R, int KR>
__device__ __forceinline__ void body(const VitTailArgs& a, const int4 me, char* smem) {
    using Tile = DuoTile<R, KR>;
    constexpr int BM = 32 * R, PA = Tile::PA, PH = Tile::PH, RP = 4 * NW, NI = BM / RP;   // RP: rows of a row phase
    constexpr int KC = NB, KO = (KR + 127) / 128;        // 16-byte chunks of a lane: of a row of x, of the attention output
    static_assert(BM % RP == 0 && NB * 128 >= 32 * NB * NW, "whole row phases, whole rows");
    bf16_t* As = (bf16_t*)smem;                         // [BM][PA]
    bf16_t* Hs = As + BM * PA;                          // [BM][PH]
    float* gs = (float*)(As + Tile::NORM);              // [2][KR]
    const int g = me.x, grow0 = me.y, slot0 = me.z, rows_g = me.w;
    const int kin = a.gt.k_in[g], de = a.gt.k_out[g], hid = a.gt.row[g];

    const int tid = threadIdx.x, w = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int l16 = tid & 15, prow = tid >> 4;          // row phases: 16 lanes a row, RP rows at a time

    // A lane's place, worked out anew by each phase that uses it: addresses that several phases share would be kept through the hidden columns,
    // in scratch, and a value from scratch is waited for like everything asked for before it.
    struct Place { int l16, prow, l32, lhi, lane; };
    auto place = [&]() __attribute__((always_inline)) {
        int t = tid;
        asm volatile("" : "+v"(t));
        return Place{t & 15, t >> 4, t & 31, (t >> 5) & 1, t & 63};
    };
    constexpr uint32_t OOB = 0x80000000u;
    const int first = ds_quotient(grow0, a.rows);                    // (of the group; rows of a tile count from there)
    auto window = [](const void* p, int64_t elements) {
        return __builtin_amdgcn_make_buffer_rsrc((void*)((const bf16_t*)p + elements), 0, 0x7fffffff, 0x00020000);
    };
    const __amdgpu_buffer_rsrc_t rx = window(a.x, (int64_t)(slot0 + first) * a.x_ss);
    uint32_t* rowx = (uint32_t*)(smem + Tile::ROWS);     // byte offset of a row of x, out of range: no such row (in LDS: not kept in registers, or in scratch)
    auto x_rows = [&](uint4 (&q)[NI][KC]) {
        const auto [l16, prow, l32, lhi, lane] = place();
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const uint32_t off = rowx[prow + RP * i] + l16 * 16;
#pragma unroll
            for (int k = 0; k < KC; ++k)
                q[i][k] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(rx, (int)((k * 16 + l16) * 8 < de ? off + k * 256 : OOB), 0, 0));
        }
    };
    // rows of C chunks a lane in the activation tile, zeros behind the slice (a chunk's last lanes may lie behind the row)
    auto to_tile = [&](const auto& q) {
        constexpr int C = sizeof(q[0]) / sizeof(uint4);
        const auto [l16, prow, l32, lhi, lane] = place();
#pragma unroll
        for (int i = 0; i < NI; ++i)
#pragma unroll
            for (int k = 0; k < C; ++k) {
                const int ch = (k * 16 + l16) * 8;
                if (128 * (k + 1) <= PA || ch < PA) *(uint4*)(As + (prow + RP * i) * PA + ch) = q[i][k];
            }
    };
    uint4 xr[NI][KC];
    {
        uint4 q[NI][KO];
        const __amdgpu_buffer_rsrc_t ro = window(a.o, (int64_t)(slot0 + first) * a.o_ss);
#pragma unroll
        for (int i = 0; i < NI; ++i) {
            const int m = grow0 + prow + RP * i, sl = ds_quotient(m, a.rows), p = m - sl * a.rows;
            const bool live = m < rows_g;
            if (l16 == 0) rowx[prow + RP * i] = live ? (uint32_t)(((sl - first) * a.x_ss + (int64_t)p * de) * 2) : OOB;
            const uint32_t ooff = live ? (uint32_t)(((sl - first) * a.o_ss + (int64_t)p * a.o_ld + l16 * 8) * 2) : OOB;
#pragma unroll
            for (int k = 0; k < KO; ++k)
                q[i][k] = __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(ro, (int)((k * 16 + l16) * 8 < kin ? ooff + k * 256 : OOB), 0, 0));
        }
        wave_sync();                                     // (a row's offset is written and read by one wavefront)
        x_rows(xr);
        for (int i = tid; i < de; i += 64 * NW) {
            gs[i] = a.g2[i];
            gs[KR + i] = a.be2[i];
        }
        to_tile(q);                                  // zeros beyond the slice
    }
    auto x_out = [&](uint32_t off, int l16, int k, const uint4& q) {     // 8 channels of a row that this thread fetched
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4_t, q), rx, (int)((k * 16 + l16) * 8 < de ? off + k * 256 : OOB), 0, 0);
    };

    // ---- acc2[b][r] += W[column block w + NW b] . act^T over K channels, 16 a step ---------------------------------------------
    f32x16_t acc2[NB][R];
    constexpr int NQ = NB < 4 ? NB : 2;                  // column blocks of Q/K/V at a time: w + NW b of every NW NQ
    constexpr std::integral_constant<int, NB> all{};
    constexpr std::integral_constant<int, NQ> some{};
    auto clear2 = [&]() {
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc2[b][r][v] = 0.f;
    };
    const uint32_t lane16 = (uint32_t)lane * 16;
    bf16x8_t ring[D];
    // Operand j of a product: step j / m of its block j % m, or step j of the one block there is.  Requests are unconditional and in a fixed order
    // (past the end of a slice they get zeros without traffic), so the number in flight is known where a product waits for the oldest; the last
    // turn of a product asks for the first operands of the next.
    struct Rows { __amdgpu_buffer_rsrc_t rs[NB]; };
    auto rows_of = [&](const Stream& t) __attribute__((always_inline)) {
        Rows v;
#pragma unroll
        for (int b = 0; b < NB; ++b) v.rs[b] = weight_row(t.n == 0 ? t.w[0] : t.w[b], 0, t.n == 0 || b < t.n ? t.k : 0);
        return v;
    };
    auto ask = [&](int j, const Rows& v, uint32_t off, bool one, int m) __attribute__((always_inline)) {
        const int so = one ? j * 1024 : j / m * 1024;
        ring[j] = __builtin_bit_cast(bf16x8_t, __builtin_amdgcn_raw_buffer_load_b128(v.rs[j % m], (int)off, so, 0));
        __builtin_amdgcn_sched_barrier(0);
    };
    auto start = [&](const Stream& t) __attribute__((always_inline)) {
        const Rows v = rows_of(t);
#pragma unroll
        for (int j = 0; j < D; ++j) ask(j, v, lane16, t.n == 0, NB);
    };
    // acc = products of N column blocks side by side (n of a stream: how many of its blocks there are; 0: the product of one block); the next
    // product has M blocks or one
    auto walk = [&](auto& acc, const Stream& t, const Stream& next, auto M, const bf16_t* act, int pitch) __attribute__((always_inline)) {
        constexpr int N = sizeof(acc) / sizeof(acc[0]), S = D / N;       // blocks, steps a turn
        static_assert(D % N == 0 && S % (N > 1 ? 2 : 4) == 0, "whole turns of whole pairs, of one block whole pairs of pairs");
        constexpr int P = 2;                             // steps that are skipped together behind the slice
        const auto [l16, prow, l32, lhi, lane] = place();
        const bf16_t* base = act + l32 * pitch + lhi * 8;
        // a pair of steps is read ahead of the products of the pair before it (one block), a step ahead of those of a step (several)
        constexpr int F = N == 1 ? 2 : 1;
        bf16x8_t f[2][F][R];
        auto read = [&](int set, int k) __attribute__((always_inline)) {
#pragma unroll
            for (int e = 0; e < F; ++e)
#pragma unroll
                for (int r = 0; r < R; ++r) f[set][e][r] = *(const bf16x8_t*)(base + r * 32 * pitch + k + e * 16);
        };
        auto product = [&](int s, int e, bool first) __attribute__((always_inline)) {
#pragma unroll
            for (int b = 0; b < N; ++b)
#pragma unroll
                for (int r = 0; r < R; ++r)
                    acc[b][r] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[(s + e) * N + b], f[s / F & 1][e][r], first ? f32x16_t{} : acc[b][r], 0, 0, 0);
        };
        const Rows mine = rows_of(t), other = rows_of(next);
        const bool one = next.n == 0;
        read(0, 0);
        int k0 = 0;
        auto turn = [&](const Rows& from, uint32_t off, bool single, int m) __attribute__((always_inline)) {
#pragma unroll
            for (int p = 0; p < S; p += P) {
                if (p == 0 || k0 + p * 16 < t.k) {       // (rows hold zeros up to whole pairs of steps)
#pragma unroll
                    for (int s = p; s < p + P; s += F) {
                        read((s / F + 1) & 1, k0 + (s + F) * 16);
                        __builtin_amdgcn_sched_barrier(0);       // (the compiler would sink the reads to their use)
                        if (s > 0) product(s, 0, false);
                        else if (k0 == 0) product(s, 0, true);
                        else product(s, 0, false);
                        if constexpr (F == 2) product(s, 1, false);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
#pragma unroll
                for (int j = p * N; j < (p + P) * N; ++j) ask(j, from, off, single, m);
            }
        };
        for (; k0 + 16 * S < t.k; k0 += 16 * S) turn(mine, lane16 + k0 * 64 + S * 1024, N == 1, N);
        turn(other, lane16, one, M.value);
    };
    // the product of a whole hidden tile (HC channels, zeros behind the slice in both operands), one piece of other work beside each of its steps
    auto walk_tile = [&](const Stream& t, const Stream& next, auto M, auto piece) __attribute__((always_inline)) {
        constexpr int S = D / NB, STEPS = HC / 16;
        const auto [l16, prow, l32, lhi, lane] = place();
        const bf16_t* base = Hs + l32 * PH + lhi * 8;
        bf16x8_t f[2][R];
        const Rows mine = rows_of(t), other = rows_of(next);
        const bool one = next.n == 0;
#pragma unroll
        for (int r = 0; r < R; ++r) f[0][r] = *(const bf16x8_t*)(base + r * 32 * PH);
#pragma unroll
        for (int s = 0; s < STEPS; ++s) {
#pragma unroll
            for (int r = 0; r < R; ++r) f[(s + 1) & 1][r] = *(const bf16x8_t*)(base + r * 32 * PH + (s + 1) * 16);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int m = 0; m < NB * R; ++m) {
                const int b = m / R, r = m % R;
                acc2[b][r] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ring[s % S * NB + b], f[s & 1][r], acc2[b][r], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
                piece(s, m);
                __builtin_amdgcn_sched_barrier(0);
            }
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                if (s + S < STEPS) ask(s % S * NB + b, mine, lane16 + (s + S) / S * (S * 1024), false, NB);
                else ask(s % S * NB + b, other, lane16, one, M.value);
            }
        }
    };
    float* line = (float*)(As + Tile::BIAS) + w * 128;
    auto columns = [&](const float* v, int c, int n) {   // n: elements of v
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc((void*)v, 0, n * 4, 0x00020000);
        return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rs, c * 4, 0, 0));
    };
    auto bias_of = [&](int b, int q) { return *(const float4*)(line + 32 * b + 8 * q + 4 * place().lhi); };
    auto to_line = [&](float v, float v2) {
        const int lane = place().lane;
        wave_sync();                                     // (what was there has been read)
        line[lane] = v;
        if constexpr (NB > 2) line[64 + lane] = v2;
        wave_sync();
    };
    // As (bf16) += acc2 + bias on the elements this lane accumulated
    auto add_columns = [&](float cst, float cst2) {
        const auto [l16, prow, l32, lhi, lane] = place();
        to_line(cst, cst2);
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            if ((w + NW * b) * 32 >= de) return;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int ch = (w + NW * b) * 32 + 8 * q + 4 * lhi;
                const float4 h = bias_of(b, q);
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    uint2* p = (uint2*)(As + (r * 32 + l32) * PA + ch);
                    const uint2 res = *p;
                    const f32x16_t& t = acc2[b][r];
                    float v0 = t[4 * q] + h.x, v1 = t[4 * q + 1] + h.y, v2 = t[4 * q + 2] + h.z, v3 = t[4 * q + 3] + h.w;
                    v0 += __uint_as_float(res.x << 16);
                    v1 += __uint_as_float(res.x & 0xffff0000u);
                    v2 += __uint_as_float(res.y << 16);
                    v3 += __uint_as_float(res.y & 0xffff0000u);
                    *p = ch < de ? make_uint2(f2bf2(v0, v1), f2bf2(v2, v3)) : make_uint2(0, 0);
                }
            }
        }
    };

    // rows of x to memory, normalised in place where it goes on: row_norm's arithmetic and order without branches (behind the slice: zeros)
    auto norm_rows = [&](bool on) __attribute__((always_inline)) {
        const auto [l16, prow, l32, lhi, lane] = place();
#pragma unroll
        for (int i0 = 0; i0 < NI; i0 += 2) {             // two rows side by side
            uint4 xq[2][KC];
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int k = 0; k < KC; ++k) {
                    const int ch = (k * 16 + l16) * 8;
                    xq[i][k] = *(const uint4*)(As + (prow + RP * (i0 + i)) * PA + ch);
                    if (128 * (k + 1) > PA && ch >= PA) xq[i][k] = make_uint4(0, 0, 0, 0);
                }
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const uint32_t off = rowx[prow + RP * (i0 + i)] + l16 * 16;
#pragma unroll
                for (int k = 0; k < KC; ++k) x_out(off, l16, k, xq[i][k]);
            }
            if (!on) continue;
            float v[2][KC][8], mu[2], rstd[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                float sum = 0.f;
#pragma unroll
                for (int k = 0; k < KC; ++k) {
                    unpack8(xq[i][k], v[i][k]);
#pragma unroll
                    for (int e = 0; e < 8; ++e) sum += v[i][k][e];
                }
                mu[i] = row16_sum(sum) / (float)de;
            }
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                float sq = 0.f;
#pragma unroll
                for (int k = 0; k < KC; ++k) {
                    const bool in = (NB > 2 && 128 * (k + 1) <= 32 * NW * (NB - 1)) || (k * 16 + l16) * 8 < de;
#pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        v[i][k][e] -= mu[i];
                        const float t = in ? v[i][k][e] : 0.f;
                        sq += t * t;
                    }
                }
                rstd[i] = 1.0f / sqrtf(row16_sum(sq) / (float)de + a.eps);
            }
#pragma unroll
            for (int k = 0; k < KC; ++k) {
                const int ch = (k * 16 + l16) * 8;
                const float4 g0 = *(const float4*)(gs + ch), g1 = *(const float4*)(gs + ch + 4);
                const float4 b0 = *(const float4*)(gs + KR + ch), b1 = *(const float4*)(gs + KR + ch + 4);
                const float gm[8] = {g0.x, g0.y, g0.z, g0.w, g1.x, g1.y, g1.z, g1.w};
                const float bt[8] = {b0.x, b0.y, b0.z, b0.w, b1.x, b1.y, b1.z, b1.w};
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    float o8[8];
#pragma unroll
                    for (int e = 0; e < 8; ++e) o8[e] = v[i][k][e] * rstd[i] * gm[e] + bt[e];
                    uint4 o = pack8(o8);
                    if (ch >= de) o = make_uint4(0, 0, 0, 0);
                    if (128 * (k + 1) <= PA || ch < PA) *(uint4*)(As + (prow + RP * (i0 + i)) * PA + ch) = o;
                }
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    const bf16_t *w1 = a.w1 + (int64_t)(w * a.kb1) * 512, *w2 = a.w2 + (int64_t)(w * a.kb2) * 512, *wp = a.wp + (int64_t)(w * a.kbp) * 512;
    const float *b1 = a.b1, *b2 = a.b2;
    int step1 = NW * a.kb1, step2 = NW * a.kb2;
    ds_hold(w1, w2, b1, b2, step1, step2);
    const int nd = (de + 31) / 32, own = nd > w ? (nd - w + NW - 1) / NW : 0;    // column blocks of the embedding, of this wavefront
    auto strided = [](const bf16_t* p, int64_t step, int k, int n) {
        return Stream{{p, p + step * 512, p + 2 * step * 512, p + 3 * step * 512}, n ? k : 0, n ? n : 1};
    };
    auto fc1 = [&](int hc) {
        const bf16_t* p = w1 + (int64_t)(hc * step1) * 512;
        return Stream{{p, p, p, p}, hid - hc * HC > w * 32 ? de : 0, 0};
    };
    auto fc2 = [&](int hc) { return strided(w2 + (int64_t)(hc * 2 * NW) * 512, step2, min(HC, hid - hc * HC), own); };
    const Stream sp = strided(wp, NW * a.kbp, kin, own);
    start(sp);
    auto both = [&](const float* v, float& c, float& c2) {
        const auto [l16, prow, l32, lhi, lane] = place();
        c = columns(v, (w + NW * lhi) * 32 + l32, de);
        if constexpr (NB > 2) c2 = columns(v, (w + NW * (2 + lhi)) * 32 + l32, de);
    };
    float cst, cst2 = 0.f;
    both(a.bp, cst, cst2);
    __syncthreads();
    walk(acc2, sp, fc1(0), all, As, PA);
    __syncthreads();                                     // every wavefront is past its last read of the attention output
    to_tile(xr);
    __syncthreads();
    add_columns(cst, cst2);
    __syncthreads();
    norm_rows(true);
    __syncthreads();

    clear2();
    const int nchunk = (hid + HC - 1) / HC;
    const bool more = (a.next >> g) & 1;
    const int nb = (kin + 31) / 32;
    auto qkv_block = [&](int p, int b, int* seg) {
        const int c = p * NW * NQ + w + NW * b;
        *seg = (c >= nb) + (c >= 2 * nb) + (c >= 3 * nb);
        return c - *seg * nb;
    };
    auto qkv = [&](int p) {
        Stream t;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            int seg;
            const int c = qkv_block(p, b < NQ ? b : 0, &seg);
            t.w[b] = a.wq + (int64_t)((seg * a.segq + c) * a.kbq) * 512;
        }
        const int left = 3 * nb - p * NW * NQ - w;       // blocks from this wavefront's first on
        t.n = more && left > 0 ? min(NQ, (left + NW - 1) / NW) : 1;
        t.k = more && left > 0 ? de : 0;
        return t;
    };
    f32x16_t acc1[1][R];
    uint2 o[4][R];                                       // hidden values of this lane, 4 a piece
    float top;                                           // half of the largest value of the lane
    auto make = [&](int hc, const Stream& next) __attribute__((always_inline)) {
        const int l32 = place().l32;
        cst = columns(b1, (hc * NW + w) * 32 + l32, hid);
        walk(acc1, fc1(hc), next, all, As, PA);
        to_line(-0.5f * cst, 0.f);                      // (see activate)
        top = 0.f;
    };
    // Part m of the NB R parts of piece s (4 consecutive columns of a row): bias, gelu_poly and rounding, the four values side by side.  One value at
    // a time is a chain of dependent instructions, and as a whole a piece would leave the matrix pipe idle.  The values are halved where sum and bias meet and
    // gelu_step starts from the halves: the same bits, where a multiplication a value at its end cost 256 images of DS-ViT 0.8 % (2145 us a pass).  (The line
    // holds minus the half bias: with a plus the compiler adds to the bias's registers and has to move the sums, 56 of them through scratch.)
    float gu[4], gv[4], gp[4];
    auto activate = [&](int s, int m) __attribute__((always_inline)) {
        constexpr int LEVELS = GELU_TERMS + 1, M = NB * R;
        const int q = s / R, r = s % R;
        f32x16_t& t = acc1[0][r];
#pragma unroll
        for (int l = m * LEVELS / M; l < (m + 1) * LEVELS / M; ++l) {
            if (l == 0) {
                const float4 h = bias_of(0, q);
                t[4 * q] = fmaf(t[4 * q], 0.5f, -h.x), t[4 * q + 1] = fmaf(t[4 * q + 1], 0.5f, -h.y);
                t[4 * q + 2] = fmaf(t[4 * q + 2], 0.5f, -h.z), t[4 * q + 3] = fmaf(t[4 * q + 3], 0.5f, -h.w);
                top = fmaxf(fmaxf(top, fabsf(t[4 * q])), fabsf(t[4 * q + 1]));
                top = fmaxf(fmaxf(top, fabsf(t[4 * q + 2])), fabsf(t[4 * q + 3]));
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) gelu_step<true>(l, t[4 * q + e], gu[e], gv[e], gp[e]);
            if (l == GELU_TERMS) {
                o[q][r] = make_uint2(f2bf2(gp[0], gp[1]), f2bf2(gp[2], gp[3]));
                asm volatile("" : "+v"(o[q][r].x), "+v"(o[q][r].y));
            }
        }
        asm volatile("" : "+v"(gp[0]), "+v"(gp[1]), "+v"(gp[2]), "+v"(gp[3]), "+v"(top));     // (here, and not where it is used)
    };
    // hidden values outside the polynomial's range (from their halves), and all of them to the tile
    auto to_hidden = [&](int hc) __attribute__((always_inline)) {
        const auto [l16, prow, l32, lhi, lane] = place();
        if (top > GELU_LIMIT / 2) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    const f32x16_t& t = acc1[0][r];
                    if (gelu_top(t[4 * q], t[4 * q + 1], t[4 * q + 2], t[4 * q + 3]) > GELU_LIMIT / 2)
                        o[q][r] = gelu_bf16x4_far<true>(o[q][r], t[4 * q], t[4 * q + 1], t[4 * q + 2], t[4 * q + 3]);
                }
        }
        if ((hc * NW + w) * 32 + 32 > hid) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if ((hc * NW + w) * 32 + 8 * q + 4 * lhi >= hid) {
#pragma unroll
                    for (int r = 0; r < R; ++r) o[q][r] = make_uint2(0, 0);
                }
        }
        __syncthreads();                                 // the previous columns have been read
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int r = 0; r < R; ++r) *(uint2*)(Hs + (r * 32 + l32) * PH + w * 32 + 8 * q + 4 * lhi) = o[q][r];
        __syncthreads();
    };
    make(0, nchunk > 1 ? fc1(1) : fc2(0));
#pragma unroll
    for (int s = 0; s < 4 * R; ++s)
#pragma unroll
        for (int m = 0; m < NB * R; ++m) activate(s, m);
    to_hidden(0);
    for (int hc = 1; hc < nchunk; ++hc) {
        make(hc, fc2(hc - 1));
        walk_tile(fc2(hc - 1), hc + 1 < nchunk ? fc1(hc + 1) : fc2(hc), all, activate);
        to_hidden(hc);
    }
    x_rows(xr);                                          // the residual rows of the last sum
    to_tile(xr);                                         // every wavefront is past its last read of the activation tile
    walk_tile(fc2(nchunk - 1), qkv(0), some, [](int, int) {});
    both(b2, cst, cst2);
    __syncthreads();
    add_columns(cst, cst2);
    if (more)
        for (int i = tid; i < de; i += 64 * NW) {
            gs[i] = a.g1[i];
            gs[KR + i] = a.be1[i];
        }
    __syncthreads();
    norm_rows(more);
    if (!more) return;
    __syncthreads();
    const auto [l16_, prow_, q32, qhi, lane_] = place();
    const bf16_t* q0 = a.qkv + (int64_t)(slot0 + first) * a.q_ss;
    uint32_t qoff[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int m = grow0 + r * 32 + q32, sl = ds_quotient(m, a.rows);
        qoff[r] = m < rows_g ? (uint32_t)(((sl - first) * a.q_ss + (int64_t)(m - sl * a.rows) * a.q_ld + 8 * qhi) * 2) : OOB;
    }
    for (int p = 0; p * NW * NQ + w < 3 * nb; ++p) {
        f32x16_t accq[NQ][R];
        int seg[4], n0[4];
#pragma unroll
        for (int b = 0; b < 4; ++b) n0[b] = qkv_block(p, b, &seg[b]) * 32;
        cst = columns(a.bq, (qhi ? seg[1] * a.q_ld + n0[1] : seg[0] * a.q_ld + n0[0]) + q32, 3 * a.q_ld);
        if constexpr (NQ > 2) cst2 = columns(a.bq, (qhi ? seg[3] * a.q_ld + n0[3] : seg[2] * a.q_ld + n0[2]) + q32, 3 * a.q_ld);
        walk(accq, qkv(p), qkv(p + 1), some, As, PA);
        to_line(cst, cst2);
#pragma unroll
        for (int b = 0; b < NQ; ++b) {
            const int nn = n0[b];
            if (seg[b] > 2) continue;
            const __amdgpu_buffer_rsrc_t rq = window(q0, (int64_t)seg[b] * a.q_seg + nn);
#pragma unroll
            for (int q = 0; q < 4; q += 2) {
                const bool in = nn + 8 * q + 8 * qhi < kin;
                const float4 h[2] = {bias_of(b, q), bias_of(b, q + 1)};
#pragma unroll
                for (int r = 0; r < R; ++r) {
                    uint32_t lo[2], hi[2];
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        const f32x16_t& t = accq[b][r];
                        const int c = 4 * (q + e);
                        lo[e] = f2bf2(t[c] + h[e].x, t[c + 1] + h[e].y);
                        hi[e] = f2bf2(t[c + 2] + h[e].z, t[c + 3] + h[e].w);
                    }
                    const auto a0 = __builtin_amdgcn_permlane32_swap(lo[0], lo[1], false, false);
                    const auto a1 = __builtin_amdgcn_permlane32_swap(hi[0], hi[1], false, false);
                    __builtin_amdgcn_raw_buffer_store_b128(u32x4_t{a0[0], a1[0], a0[1], a1[1]}, rq, (int)(in ? qoff[r] + 16 * q : OOB), 0, 0);
                }
            }
        }
    }
}

template <int R, int KR>
__global__ __launch_bounds__(64 * NW, 2) void vit_duo_kernel(const VitTailArgs a) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int4 me = ds_tile_record_of(a.offsets, a.gt.T, a.rows, (int)blockIdx.x, 32 * R);
    if (me.x < 0) return;
    const int de = a.gt.k_out[me.x];
    if (de <= 0) return;
    if (de <= 64 * NW) body<2, 16, R, KR>(a, me, smem);
    else if (KR <= 96 * NW || de <= 96 * NW) body<3, 12, R, KR>(a, me, smem);
    else if constexpr (KR > 96 * NW) body<4, 8, R, KR>(a, me, smem);
}

template <int KR>
int32_t launch(const VitTailArgs& a, int64_t tiles, hipStream_t s) {
    constexpr int SMEM = DuoTile<2, KR>::SMEM;
    const int32_t rc = ds_reserve_lds((const void*)vit_duo_kernel<2, KR>, SMEM, "transformer block tail");
    if (rc) return rc;
    ProfScope prof(DS_K_TAIL, s);
    hipLaunchKernelGGL((vit_duo_kernel<2, KR>), dim3((unsigned)tiles), dim3(64 * NW), SMEM, s, a);
    DS_CHECK_LAUNCH("transformer block tail");
    return DS_OK;
}

}  // namespace

int32_t ds_launch_vit_duo(const VitTailArgs& a, int64_t tiles, int width, hipStream_t s) {
    return width > 384 ? launch<416>(a, tiles, s) : launch<384>(a, tiles, s);
}
