// The first three layers of the separable networks in one kernel: 3x3 stride-2 stem convolution of the image, the first
// depthwise-separable block at stride 1 and the second at stride 2 (N x N depthwise filters, N = 3 or 5, each layer with
// batch-norm and ReLU; Section 3.2, Eq. 9 and 10).  Apart, they write and read the two largest maps of the network.
//
// A workgroup of four wavefronts goes down a strip of 14 or 28 output columns, two map rows (one output row) a turn, with the
// last rows of both maps in LDS rings.  Rows are kept from turn to turn, so only the columns on either side of a strip are
// computed twice (32 map columns for 28, 64 for 56).  A turn has two halves, each ended by a barrier:
//   depthwise   both depthwise layers, filter rows as band matrices (band.h), into operand tiles [pixel][channel];
//   products    stem, first and second pointwise layer on v_mfma_f32_16x16x32_bf16.  Stem and first pointwise layer have pixels
//               as the row operand, so a lane ends with four neighbouring pixels of a channel, as the next depthwise layer
//               reads them; the second has filters there and stores eight channels of a pixel.
// The layers of a half work on different rows (the stem is a turn ahead of the first block, which is one ahead of the second),
// so nothing in it waits for another; every wavefront has the same share of each layer, its filters in registers.
// A strip is cut into bands of rows where there are few samples, and where the last generation of workgroups would be nearly
// empty; a band computes the rows above it again and sets up its own filters (5 us).
//
// Us, three launches before (stem_mfma_kernel, bandpw_kernel twice) -> here (what reading the images and writing the output
// takes at the 5.1 TB/s of a large copy): DS-MBNet 256 images 66 + 134 + 148 -> 170 (55), one image 4.9 + 5.6 + 5.1 -> 9.6;
// DS-MBNet++ 96 images 20 + 33 + 25 -> 46 (14).  Bound by the instructions of a turn: one workgroup in a compute unit takes 1.15
// us a turn, three take 1.8, about 0.6 each.  162 registers hold it at three workgroups; held to 128 for four of them it
// spills: 261 us.  With each ring row's place a constant (six turns laid out one behind the other) a turn has a third fewer
// instructions and took no less time (189 us, 34 KB of code).
//
// Operands, fp32 sums and roundings are the three launches'; the stem, both pointwise layers and the second depthwise layer give the same bits.
// In the first depthwise layer the strips of four outputs start P columns left of an even column, so the taps of a filter row fall into
// other steps of v_mfma_f32_4x4x4 and a sum can end a last bit away: alone it changes 4 of 25.7e6 values behind it (3x3 filters, 64
// images) and 9 of 9.6e6 (5x5).
#include <algorithm>
#include <type_traits>

#include "band.h"

namespace {

struct FrontArgs {
    const bf16_t* img;            // [B][3][H][W]
    bf16_t* y;                    // [B][H2][W2][F]
    const bf16_t *ws, *wd0, *wp0, *wd1, *wp1;   // [27][C0]; [KS0][KS0][C0]; operand tiles; [KS1][KS1][C1]; operand tiles
    const float *ss, *hs, *sd0, *hd0, *sp0, *hp0, *sd1, *hd1, *sp1, *hp1;
    int32_t F, H, W, H1, W1, H2, W2, KS0, KS1, B;
    int32_t TW, strips, bands, band_rows, slots;
};

// N: depthwise filter; G0, G1: groups of 16 channels of the two maps; FP: groups of 32 filters of the second block; NT: tiles of
// 16 columns of a map row
template <int N, int G0, int G1, int FP, int NT>
struct Front {
    static constexpr int P = (N - 1) / 2, NO = NT / 2, TW = (16 * NT - 2 * N + 3) / 2;
    static constexpr int ROW = NT * 32, RS = N + 1, RM = N;             // bytes of a channel's map row; rows of the rings
    // LDS, for 64 banks: a channel's rows 8 dwords further round than the channel's before it (8 channels x 4 quads a read of the
    // first map), or 16 or 48, and 2 more every 4 channels (every other quad of the second); operand rows 4 dwords further than
    // their channels; image rows and channels so that four (channel, row) pairs of a product lie 16 dwords apart
    static constexpr int PITCH0 = NT == 2 ? 288 : 800, PITCH1 = NT == 2 ? 192 : 704;
    static constexpr int LD0 = 80, CK1 = G1 * 16, LD1 = CK1 * 2 + 16;   // bytes of an operand row: 32 channels, G1 * 16 channels
    static constexpr int PQ = 8 * NT + 1, PIECES = 15 * PQ, NL = (PIECES + 255) / 256;   // image: 3 x 5 rows of 4-pixel pieces
    static constexpr int IROW = NT == 2 ? 160 : 288, ICH = NT == 2 ? 992 : 1632;
    static constexpr int MAP0 = G0 * 16 * PITCH0 + 64, MAP1 = G1 * 16 * PITCH1 + G1 * 4 * 8 + 64;
    static constexpr int OP0 = 2 * NT * 16 * LD0, OP1 = NO * 16 * LD1, IMG = 3 * ICH, TAB = FP * 32 * 8;
    static constexpr int SMEM = MAP0 + MAP1 + OP0 + OP1 + IMG + TAB;
    static constexpr int F0 = band_filter_pitch(N, 1), F1 = band_filter_pitch(N, 2);     // while the bands are made
    static constexpr int AT_ONCE = std::min(3, 160 * 1024 / SMEM);
    static_assert(G0 * NT == 4 && G1 * NO == 4 && NO * FP == 4 && G0 * 16 * F0 + G1 * 16 * F1 <= SMEM, "equal shares");
};

template <int N, int G0, int G1, int FP, int NT>
__global__ __launch_bounds__(256, (Front<N, G0, G1, FP, NT>::AT_ONCE)) void front_kernel(const FrontArgs a) {
    using K = Front<N, G0, G1, FP, NT>;
    constexpr int P = K::P, C0 = G0 * 16, C1 = G1 * 16, SM = NT / 2, ROW = K::ROW, RS = K::RS, RM = K::RM, CK1 = K::CK1, KT1 = CK1 / 32, NL = K::NL, PQ = K::PQ, LD0 = K::LD0, LD1 = K::LD1;
    constexpr int T0 = band_steps(N, 1), T1 = band_steps(N, 2);
    extern __shared__ __attribute__((aligned(16))) char smem[];
    char *const map0 = smem, *const map1 = map0 + K::MAP0, *const op0 = map1 + K::MAP1, *const op1 = op0 + K::OP0, *const image = op1 + K::OP1;
    float* const tab = (float*)(image + K::IMG);                  // [FP * 32] scale, then shift of the second block's filters
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), l16 = lane & 15, kg = lane >> 4;
    const int slot = blockIdx.x % a.slots, rest = blockIdx.x / a.slots, strip = rest % a.strips, band = rest / a.strips;
    if (slot >= a.B) return;
    const int x0 = strip * a.TW, t0 = band * a.band_rows, t1 = min(a.H2, t0 + a.band_rows);
    if (t0 >= t1) return;
    const int u0 = t0 - P, v0 = u0 - P;

    // ---- image pieces: rows 4 v + 4 P - 3 .. + 1 of each channel, from column 4 x0 - 4 P - 4 on ----
    int poff[NL], pcol[NL], prow[NL], plds[NL];
#pragma unroll
    for (int i = 0; i < NL; ++i) {
        const int c = tid + 256 * i, row = c / PQ, q = c - row * PQ, ch = row / 5;
        pcol[i] = 4 * x0 - 4 * P - 4 + 4 * q;
        prow[i] = c < K::PIECES && pcol[i] >= 0 && pcol[i] + 3 < a.W ? row - ch * 5 : 0x20000000;
        plds[i] = ch * K::ICH + (row - ch * 5) * K::IROW + q * 8;
        poff[i] = ((ch * a.H + row - ch * 5) * a.W + pcol[i]) * 2;
    }
    const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc((void*)(a.img + (int64_t)slot * 3 * a.H * a.W), 0, 3 * a.H * a.W * 2, 0x00020000);
    uint2 pix[NL];
    const auto fetch = [&](int v) {
        const int r0 = 4 * v + 4 * P - 3;
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            const auto t = __builtin_amdgcn_raw_buffer_load_b64(xr, (unsigned)(prow[i] + r0) < (unsigned)a.H ? poff[i] + r0 * a.W * 2 : (int)BAND_OOB, 0, 0);
            pix[i] = make_uint2(t[0], t[1]);
        }
    };
    fetch(v0);

    // ---- what stays in registers ----
    // stem: reduction order (channel, row) pairs x four columns, the first of them under a zero weight
    const int row = wave >> 1, tile = (wave & 1) * SM;            // of the stem's and the first pointwise layer's SM tiles
    typedef __attribute__((ext_vector_type(8))) short short8_t;
    short8_t sw[G0][2];
    float ssc[G0], ssh[G0];
#pragma unroll
    for (int g = 0; g < G0; ++g) {
        const auto w = [&](int pair, int e) { return e ? (short)a.ws[((pair % 3 * 3 + e - 1) * 3 + pair / 3) * C0 + g * 16 + l16] : (short)0; };
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            sw[g][0][k] = w(kg * 2 + (k >> 2), k & 3);
            sw[g][1][k] = k < 4 && !kg ? w(8, k & 3) : (short)0;
        }
        ssc[g] = a.ss[g * 16 + l16];
        ssh[g] = a.hs[g * 16 + l16];
    }
    // depthwise: this lane's channels, strips of four outputs
    const int b = lane >> 2, d0c = wave % G0 * 16 + b, d0g = wave / G0, d1c = wave % G1 * 16 + b, d1g = wave / G1;
    const bool odd = b & 1;
    const int st = odd ? 3 - (lane & 3) : lane & 3;
    const float d0s = a.sd0[d0c], d0h = a.hd0[d0c], d1s = a.sd1[d1c], d1h = a.hd1[d1c];
    // pointwise
    constexpr int kb0 = (C0 + 31) / 32 | 1, kb1 = (C1 + 31) / 32 | 1;
    const int n0 = (l16 >> 2) * 8 + (l16 & 3), p1g = wave % FP, p1t = wave / FP, n1 = p1g * 32 + kg * 8;
    bf16x8_t w0[G1];
    float p0s[G1], p0h[G1];
#pragma unroll
    for (int g = 0; g < G1; ++g) {
        w0[g] = *(const bf16x8_t*)((const char*)a.wp0 + (g >> 1) * kb0 * 2048 + (g & 1) * 1024 + lane * 16);
        p0s[g] = a.sp0[(g >> 1) * 32 + (g & 1) * 4 + n0];
        p0h[g] = a.hp0[(g >> 1) * 32 + (g & 1) * 4 + n0];
    }
    bf16x8_t w1[KT1][2];
#pragma unroll
    for (int k = 0; k < KT1; ++k)
#pragma unroll
        for (int h = 0; h < 2; ++h)
            w1[k][h] = *(const bf16x8_t*)((const char*)a.wp1 + (p1g * 32 < a.F ? (p1g * kb1 + k) * 2048 + h * 1024 : 0) + lane * 16);
    // the bands, from filters laid out between zeros; everything is asked for before anything is waited for
    constexpr int TAPS = (C0 + C1) * N * N, NF = (TAPS + 255) / 256;
    const int k0 = (a.KS0 - N) / 2, k1 = (a.KS1 - N) / 2;
    bf16_t tap[NF];
    int spot[NF];
#pragma unroll
    for (int h = 0; h < NF; ++h) {
        const int e = min(tid + h * 256, TAPS - 1), t = e / (C0 + C1), c = e - t * (C0 + C1), i = t / N, j = t - i * N;
        const bool second = c >= C0;
        tap[h] = second ? a.wd1[((k1 + i) * a.KS1 + k1 + j) * C1 + c - C0] : a.wd0[((k0 + i) * a.KS0 + k0 + j) * C0 + c];
        spot[h] = second ? C0 * K::F0 + (c - C0) * K::F1 + (i * band_row_dwords(2) * 2 + band_lead(2) + j) * 2
                         : c * K::F0 + (i * band_row_dwords(1) * 2 + band_lead(1) + j) * 2;
    }
    const float tsc = a.sp1[min(tid, a.F - 1)], tsh = a.hp1[min(tid, a.F - 1)];
    for (int e = tid; e < K::SMEM / 16; e += 256) ((uint4*)smem)[e] = make_uint4(0, 0, 0, 0);
    __syncthreads();
#pragma unroll
    for (int h = 0; h < NF; ++h) *(bf16_t*)(smem + spot[h]) = tap[h];
    __syncthreads();
    short4_t A0[N][T0], A1[N][T1];
    band_operand<N, 1>(A0, smem + d0c * K::F0);
    band_operand<N, 2>(A1, smem + G0 * 16 * K::F0 + d1c * K::F1);
    __syncthreads();
    for (int e = tid; e < K::SMEM / 16; e += 256) ((uint4*)smem)[e] = make_uint4(0, 0, 0, 0);
    __syncthreads();
    if (tid < a.F) {
        tab[tid] = tsc;
        tab[FP * 32 + tid] = tsh;
    }

    // masks of this lane's four pixels of a tile: columns outside the maps are the next layer's padding, zeros
    const auto mask = [](int x, int w) {
        return make_uint2(((unsigned)x < (unsigned)w ? 0xffffu : 0u) | ((unsigned)(x + 1) < (unsigned)w ? 0xffff0000u : 0u),
                          ((unsigned)(x + 2) < (unsigned)w ? 0xffffu : 0u) | ((unsigned)(x + 3) < (unsigned)w ? 0xffff0000u : 0u));
    };
    uint2 ms[SM], mp[SM];
#pragma unroll
    for (int j = 0; j < SM; ++j) {
        ms[j] = mask(2 * x0 - 2 * P + (tile + j) * 16 + kg * 4, a.W1);
        mp[j] = mask(2 * x0 - P + (tile + j) * 16 + kg * 4, a.W1);
    }
    // four pixels of a channel: batch-norm, ReLU (0 for NaN)
    const auto finish = [](f32x4_t d, float sc, float sh) {
        return make_uint2(f2bf2(fmaxf(d[0] * sc + sh, 0.f), fmaxf(d[1] * sc + sh, 0.f)), f2bf2(fmaxf(d[2] * sc + sh, 0.f), fmaxf(d[3] * sc + sh, 0.f)));
    };
    const __amdgpu_buffer_rsrc_t yr = __builtin_amdgcn_make_buffer_rsrc((void*)(a.y + (int64_t)slot * a.H2 * a.W2 * a.F), 0, a.H2 * a.W2 * a.F * 2, 0x00020000);
    const int yoff = p1t * 16 + l16 < a.TW && x0 + p1t * 16 + l16 < a.W2 && n1 < a.F ? (x0 + p1t * 16 + l16) * a.F * 2 + n1 * 2 : (int)BAND_OOB;
    // addresses of this lane
    const char* const d0p = map0 + d0c * K::PITCH0 + (d0g * 4 + st) * 8;
    const char* const d1p = map1 + d1c * K::PITCH1 + (d1c >> 2) * 8 + (d1g * 4 + st) * 16;
    char* const sp = map0 + l16 * K::PITCH0 + tile * 32 + kg * 8;
    char* const pp = map1 + n0 * K::PITCH1 + (n0 >> 2) * 8 + tile * 32 + kg * 8;
    char* const d0o = op0 + (d0g * 16 + st * 4 + (odd ? 2 : 0)) * LD0 + (d0c & ~1) * 2;
    char* const d1o = op1 + (d1g * 16 + st * 4 + (odd ? 2 : 0)) * LD1 + (d1c & ~1) * 2;
    const char* const p0o = op0 + ((row * NT + tile) * 16 + l16) * LD0 + kg * 16;
    const char* const p1o = op1 + (p1t * 16 + l16) * LD1 + kg * 16;
    const auto pair = [](int p) { return p / 3 * K::ICH + p % 3 * K::IROW; };
    const char* const sx = image + row * 2 * K::IROW + (tile * 16 + l16) * 4 + 4;
    const char *const sa = sx + pair(kg * 2), *const sb = sx + pair(kg * 2 + 1);

    // Turn i of the strip, counted from v0 - 1: its rows in the rings are constants of the turn's number modulo their sizes.
    // inner: every layer has a row, all of them inside their maps
    const auto turn = [&](auto inner_, int i, int n) __attribute__((always_inline)) {
        constexpr bool inner = decltype(inner_)::value;
        const int rs = 2 * n % RS, rd = 2 * (n + RS - P - 1) % RS, rp = 2 * (n + RM - P - 1) % RM, rm = (1 + 2 * (n + 2 * RM - 2 * P - 2)) % RM;
        const bool stem = inner || i + 1 < t1, first = inner || (i >= u0 && i < t1), second = inner || i > t0;
        // ---- image rows of the next turn, depthwise layers ----
        const auto at0 = [rd](int r) { return (rd + r) % RS * ROW; };
        const auto at1 = [rm](int r) { return (rm + r) % RM * ROW; };
        f32x4_t e0[2], e1[1];
        uint2 o0[2], o1[1];
        float chk = 0.f;
        const auto put0 = [&] {
#pragma unroll
            for (int y = 0; y < 2; ++y) {
                const uint2 t = band_trade(o0[y], odd);
                *(uint32_t*)(d0o + y * NT * 16 * LD0) = t.x;
                *(uint32_t*)(d0o + y * NT * 16 * LD0 + LD0) = t.y;
            }
        };
        const auto put1 = [&] {
            const uint2 t = band_trade(o1[0], odd);
            *(uint32_t*)d1o = t.x;
            *(uint32_t*)(d1o + LD1) = t.y;
        };
        if (stem) {
#pragma unroll
            for (int h = 0; h < NL; ++h)
                if (tid + 256 * h < K::PIECES) *(uint2*)(image + plds[h]) = pix[h];
            if (inner || i + 2 < t1) fetch(i + 2);
        }
        if (first) {
            band_rows_at<N, 1, 2>(e0, A0, d0p, at0);
            chk = band_finish<2>(o0, e0, d0s, d0h, true);
            put0();
        }
        if (second) {
            band_rows_at<N, 2, 1>(e1, A1, d1p, at1);
            const float c = band_finish<1>(o1, e1, d1s, d1h, true);
            chk = chk != 0.f ? chk : c;
            put1();
        }
        if (__ballot(chk != 0.f)) {
            if (first) {
                if (chk != 0.f) band_exact_at<N, 1, 2>(o0, d0s, d0h, true, [&](int r, int c) { return a.wd0[((k0 + r) * a.KS0 + k0 + c) * C0 + d0c]; }, d0p, at0);
                put0();
            }
            if (second) {
                if (chk != 0.f) band_exact_at<N, 2, 1>(o1, d1s, d1h, true, [&](int r, int c) { return a.wd1[((k1 + r) * a.KS1 + k1 + c) * C1 + d1c]; }, d1p, at1);
                put1();
            }
        }
        __syncthreads();
        // ---- products ----
        const f32x4_t none = {0.f, 0.f, 0.f, 0.f};
        // four pixels a lane, into a ring row; columns outside the map are zeros
        const auto put = [&](char* q, f32x4_t d, float sc, float sh, uint2 m, bool ok) __attribute__((always_inline)) {
            const uint2 o = finish(d, sc, sh);
            *(uint2*)q = ok ? make_uint2(o.x & m.x, o.y & m.y) : make_uint2(0, 0);
        };
        if (stem) {
            char* const q = sp + (rs + row) * ROW;
            const bool ok = inner || (unsigned)(2 * i + 1 + 2 * P + row) < (unsigned)a.H1;
#pragma unroll
            for (int j = 0; j < SM; ++j) {
                const uint4 lo = make_uint4(*(const uint32_t*)(sa + j * 64), *(const uint32_t*)(sa + j * 64 + 4), *(const uint32_t*)(sb + j * 64), *(const uint32_t*)(sb + j * 64 + 4));
                const uint2 t = make_uint2(*(const uint32_t*)(sx + pair(8) + j * 64), *(const uint32_t*)(sx + pair(8) + j * 64 + 4));
                const uint4 hi = make_uint4(kg ? 0u : t.x, kg ? 0u : t.y, 0u, 0u);
                f32x4_t d[G0];
#pragma unroll
                for (int g = 0; g < G0; ++g) d[g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, lo), __builtin_bit_cast(bf16x8_t, sw[g][0]), none, 0, 0, 0);
#pragma unroll
                for (int g = 0; g < G0; ++g) d[g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, hi), __builtin_bit_cast(bf16x8_t, sw[g][1]), d[g], 0, 0, 0);
#pragma unroll
                for (int g = 0; g < G0; ++g) put(q + g * 16 * K::PITCH0 + j * 32, d[g], ssc[g], ssh[g], ms[j], ok);
            }
        }
        if (first) {
            char* const q = pp + (row ? (rp + 1) % RM : rp) * ROW;
            const bool ok = inner || (unsigned)(2 * i + P - 1 + row) < (unsigned)a.H1;
#pragma unroll
            for (int j = 0; j < SM; ++j) {
                const bf16x8_t f = *(const bf16x8_t*)(p0o + j * 16 * LD0);
                f32x4_t d[G1];
#pragma unroll
                for (int g = 0; g < G1; ++g) d[g] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(f, w0[g], none, 0, 0, 0);
#pragma unroll
                for (int g = 0; g < G1; ++g)                                 // filters 4 and 32 on
                    put(q + (g & 1) * (4 * K::PITCH1 + 8) + (g >> 1) * (32 * K::PITCH1 + 64) + j * 32, d[g], p0s[g], p0h[g], mp[j], ok);
            }
        }
        f32x4_t d1[2] = {none, none};
        if (second) {
#pragma unroll
            for (int k = 0; k < KT1; ++k) {
                const bf16x8_t f = *(const bf16x8_t*)(p1o + k * 64);
#pragma unroll
                for (int h = 0; h < 2; ++h) d1[h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w1[k][h], f, d1[h], 0, 0, 0);
            }
        }
        if (second) {
            float v[8];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const float4 sc = *(const float4*)(tab + n1 + 4 * h), sh = *(const float4*)(tab + FP * 32 + n1 + 4 * h);
                v[4 * h] = fmaxf(d1[h][0] * sc.x + sh.x, 0.f);
                v[4 * h + 1] = fmaxf(d1[h][1] * sc.y + sh.y, 0.f);
                v[4 * h + 2] = fmaxf(d1[h][2] * sc.z + sh.z, 0.f);
                v[4 * h + 3] = fmaxf(d1[h][3] * sc.w + sh.w, 0.f);
            }
            typedef __attribute__((ext_vector_type(4))) uint32_t u4;
            const u4 r = {f2bf2(v[0], v[1]), f2bf2(v[2], v[3]), f2bf2(v[4], v[5]), f2bf2(v[6], v[7])};
            __builtin_amdgcn_raw_buffer_store_b128(r, yr, yoff, (i - 1) * a.W2 * a.F * 2, 0);
        }
        __syncthreads();
    };
    const int end = min(t1 - 2, (a.H1 - 1 - 2 * P) / 2);                     // inner turns lie below it
    for (int i = v0 - 1, n = 0; i <= t1; ++i, ++n) {
        if (i > t0 && i < end) turn(std::true_type{}, i, n);
        else turn(std::false_type{}, i, n);
    }
}

template <int N, int G0, int G1, int FP, int NT>
int32_t launch(FrontArgs& a, hipStream_t s) {
    using K = Front<N, G0, G1, FP, NT>;
    a.strips = (a.W2 + K::TW - 1) / K::TW;
    a.TW = (a.W2 + a.strips - 1) / a.strips;
    a.slots = a.B >= 32 ? (a.B + 7) & ~7 : a.B;            // a sample's strips on one die where that costs few empty slots
    // bands: the fewest turns, counting those above a band's first row and what a workgroup sets up
    int64_t best = INT64_MAX;
    for (int n = 1; n <= a.H2; ++n) {
        const int rows = (a.H2 + n - 1) / n;
        const int64_t rounds = ((int64_t)a.B * a.strips * n + 256 * K::AT_ONCE - 1) / (256 * K::AT_ONCE), turns = rounds * (rows + N + 2);
        if (turns < best) {
            best = turns;
            a.band_rows = rows;
        }
    }
    a.bands = (a.H2 + a.band_rows - 1) / a.band_rows;
    const int64_t grid = (int64_t)a.slots * a.strips * a.bands;
    if (grid > 0x3fffffff) return DS_EUNSUPPORTED;
    const int32_t rc = ds_reserve_lds((const void*)front_kernel<N, G0, G1, FP, NT>, K::SMEM, "first layers");
    if (rc) return rc;
    ProfScope prof(DS_K_DWCONV, s);
    hipLaunchKernelGGL((front_kernel<N, G0, G1, FP, NT>), dim3((unsigned)grid), dim3(256), K::SMEM, s, a);
    DS_CHECK_LAUNCH("stem and first two separable blocks");
    return DS_OK;
}

}  // namespace

int32_t ds_launch_front(const bf16_t* img, int32_t B, int32_t H, int32_t W, const FrontLayers& l, bf16_t* y, hipStream_t s) {
    if (B <= 0) return DS_OK;
    const int H1 = (H - 1) / 2 + 1, W1 = (W - 1) / 2 + 1, H2 = (H1 - 1) / 2 + 1, W2 = (W1 - 1) / 2 + 1;
    const int n = l.taps;
    if (W % 4 || l.F % 8 || l.F < 8 || l.KS0 < n || l.KS1 < n || (l.KS0 - n) % 2 ||
        (l.KS1 - n) % 2 || (int64_t)3 * H * W * 2 >= 0x7fffffffLL || (int64_t)H2 * W2 * l.F * 2 >= 0x7fffffffLL)
        return DS_EUNSUPPORTED;
    FrontArgs a = {};
    a.img = img; a.y = y; a.ws = l.ws; a.wd0 = l.wd0; a.wp0 = l.wp0; a.wd1 = l.wd1; a.wp1 = l.wp1;
    a.ss = l.ss; a.hs = l.hs; a.sd0 = l.sd0; a.hd0 = l.hd0; a.sp0 = l.sp0; a.hp0 = l.hp0;
    a.sd1 = l.sd1; a.hd1 = l.hd1; a.sp1 = l.sp1; a.hp1 = l.hp1;
    a.F = l.F; a.KS0 = l.KS0; a.KS1 = l.KS1;
    a.H = H; a.W = W; a.H1 = H1; a.W1 = W1; a.H2 = H2; a.W2 = W2; a.B = B;
    if (n == 3 && l.C0 == 32 && l.C1 == 64 && l.F <= 128) return launch<3, 2, 4, 4, 2>(a, s);
    if (n == 5 && l.C0 == 16 && l.C1 == 32 && l.F <= 64) return launch<5, 1, 2, 2, 4>(a, s);
    return DS_EUNSUPPORTED;
}
