// Depthwise-separable block of the layers in front of the gate (one group, full width) in one kernel: N x N depthwise
// convolution (N = 3 or 5, padding (N - 1) / 2, stride 1 or 2) + batch-norm + ReLU feeding the 1x1 pointwise convolution +
// batch-norm + ReLU (Section 3.2, Eq. 9 and 10; 11 and 13 with a cropped filter).  The depthwise map stays in the compute unit.
//
// The maps in front of the gate are the largest of the network and both layers are thin, so memory is the bound; what the
// two layers apart, and a workgroup per tile, lose is the map in between and every tile's chain of load, depthwise, product
// and store.  A workgroup here stays, goes over tiles of RO rows x up to 16 columns (PT at a time), and has the next tile's
// pixels on their way from the moment that the present ones are in LDS; both layers' filters stay in registers and LDS.
// 7 rows at stride 1, 4 at stride 2.  256 images (both layers before -> here; what moving input and output once takes at the
// 5.1 TB/s of a large copy; profiles/layers_mbnet_b256.txt, layers_mbnet_pp_b96.txt):
//   112x112, 32 -> 64                  141 -> 135 (121) us      112x112, 64 -> 128, stride 2   143 -> 148 (121)
//   56x56, 128 -> 128                  134 ->  95 (81)          56x56, 128 -> 256, stride 2     88 ->  70 (60)
//   28x28, 256 -> 256                  102 ->  64 (40)
// and for 5x5 filters, 96 images: 112x112, 16 -> 32 70 -> 34 (23); 112x112, 32 -> 48, stride 2 41 -> 25 (21); 56x56, 48 -> 48
// 44 -> 22 (11).  The thinnest layers are bound by the vector instructions around the products (batch-norm, packing).
//   windows       pixels x channels of a chunk (16 NW / PT channels), by channel, in LDS;
//   depthwise     a wavefront takes 16 channels of a tile: filter rows as band matrices (band.h), batch-norm, ReLU, bf16 into
//                 the operand tile [pixel][channel];
//   pointwise     a wavefront takes 32 NP filters of a tile: v_mfma_f32_16x16x32_bf16, each row a column operand.
#include <algorithm>

#include "band.h"

namespace {

constexpr int STRIPS = 4;

struct BandPwArgs {
    const bf16_t* x;              // [B][H][W][C]
    bf16_t* y;                    // [B][H][W][F]
    const bf16_t *wd, *wp;        // [KS][KS][C]; operand tiles (see the header)
    const float *sd, *hd, *sp, *hp;
    int32_t KS, C, F, H, W, Ho, Wo, B, kb;
    int32_t TW, xtiles, tiles, tsets, slots, items;
};

// 16-byte octet of an operand row of CK channels, turned by the pixel so that 8 or 16 neighbouring pixels' octets of one
// channel octet meet every bank once
template <int CK>
__device__ __forceinline__ int turn(int octet, int px) {
    return octet ^ (CK >= 128 ? px & 15 : CK == 64 ? px & 7 : (px >> 1) & 3);
}

// KT: steps of 32 channels.  Every workgroup has the same number of items, give or take one, so all end together
template <int N, int S, int NW, int PT, int KT, int NP>
struct BandPw {
    static constexpr int WT = NW / PT, CK = 16 * WT, CHUNKS = (KT * 32 + CK - 1) / CK, KS = CK / 32;
    static constexpr int RO = S == 1 ? 7 : 4, PX = RO * 16, ROWS = (RO - 1) * S + N, NQ = band_quads(STRIPS, N, S), PITCH = band_pitch(ROWS, NQ), WIN = band_window(CK, PITCH);
    static constexpr int FP = band_filter_pitch(N, S), FLT = (CHUNKS * 16 * FP + 15) & ~15;
    static constexpr int OCT = CK / 8, TASKS = ROWS * NQ * OCT, NT = (TASKS + WT * 64 - 1) / (WT * 64);
    static constexpr int SMEM = PT * PX * CK * 2 + PT * WIN + NW * FLT;
    static constexpr int AT_ONCE = NW == 4 ? (KT == 1 && 3 * SMEM <= 160 * 1024 ? 3 : 2) : 1;   // workgroups in a compute unit
};

template <int N, int S, int NW, int PT, int KT, int NP>
__global__ __launch_bounds__(NW * 64, (NW == 4 ? BandPw<N, S, NW, PT, KT, NP>::AT_ONCE : 2)) void bandpw_kernel(const BandPwArgs a) {
    using K = BandPw<N, S, NW, PT, KT, NP>;
    constexpr int WT = K::WT, CK = K::CK, CHUNKS = K::CHUNKS, RO = K::RO, MF = RO, PX = K::PX, NQ = K::NQ, PITCH = K::PITCH, WIN = K::WIN, FP = K::FP, NT = K::NT, OCT = K::OCT;
    constexpr bool HOLD = KT <= 4 && CHUNKS * N * band_steps(N, S) <= 15;                        // the bands fit beside the rest
    extern __shared__ __attribute__((aligned(16))) char smem[];   // operand tiles, windows, each wavefront's depthwise filters
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int sub = wave % WT, own = wave / WT;                   // of the own tile
    char* const ops = smem + own * (PX * CK * 2);
    char* const win = smem + PT * PX * CK * 2;
    char* const flt = win + PT * WIN + wave * K::FLT;
    const int b = lane >> 2, cl = sub * 16 + b, kg = lane >> 4;
    const bool odd = b & 1;
    const int st = odd ? 3 - (lane & 3) : lane & 3;

    // what stays: the depthwise filters between zeros and their batch-norm, the pointwise filters in operand order
    for (int e = lane; e < K::FLT / 16; e += 64) ((uint4*)flt)[e] = make_uint4(0, 0, 0, 0);
    __syncthreads();
    const int k0 = (a.KS - N) / 2;
    for (int e = lane; e < CHUNKS * N * N * 2; e += 64) {
        const int c8 = e & 1, t = (e >> 1) % (N * N), q = (e >> 1) / (N * N), i = t / N, ch = q * CK + sub * 16 + c8 * 8;
        const uint4 v = *(const uint4*)(a.wd + (int64_t)((k0 + i) * a.KS + k0 + t - i * N) * a.C + min(ch, a.C - 8));
        bf16_t* p = (bf16_t*)(flt + (q * 16 + c8 * 8) * FP) + i * band_row_dwords(S) * 2 + band_lead(S) + t - i * N;
        const uint32_t* u = &v.x;
#pragma unroll
        for (int k = 0; k < 8; ++k) p[k * (FP / 2)] = (bf16_t)(u[k / 2] >> (k & 1) * 16);
    }
    float sc[CHUNKS], sh[CHUNKS];                                 // zeros past the last channel, which makes its map zeros
#pragma unroll
    for (int q = 0; q < CHUNKS; ++q) {
        sc[q] = q * CK + cl < a.C ? a.sd[q * CK + cl] : 0.f;
        sh[q] = q * CK + cl < a.C ? a.hd[q * CK + cl] : 0.f;
    }
    float s[NP][8], t[NP][8];
#pragma unroll
    for (int j = 0; j < NP; ++j)
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            const int n = min((sub + WT * j) * 32 + kg * 8, a.F - 8) + k;
            s[j][k] = a.sp[n];
            t[j][k] = a.hp[n];
        }
    bf16x8_t wf[NP][KT][2];
#pragma unroll
    for (int j = 0; j < NP; ++j)
#pragma unroll
        for (int k = 0; k < KT; ++k)
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const int grp = sub + WT * j;
                const bool ok = grp * 32 < a.F && k < a.kb;
                wf[j][k][h] = *(const bf16x8_t*)((const char*)a.wp + (ok ? (grp * a.kb + k) * 2048 + h * 1024 : 0) + lane * 16);
            }

    // loads: quads of 4 pixels x 8 channels of the tile's window, dealt to its lanes with the channels fastest
    const int oct = threadIdx.x % OCT, px2 = a.C * 2;
    int prow[NT], pcol[NT], poff[NT], plds[NT];
#pragma unroll
    for (int h = 0; h < NT; ++h) {
        const int q = (threadIdx.x % (WT * 64) + h * WT * 64) / OCT, row = q / NQ;
        prow[h] = q < K::ROWS * NQ ? row : 0x40000000;
        pcol[h] = (q - row * NQ) * 4;
        poff[h] = (row * a.W + pcol[h]) * px2 + oct * 16;
        plds[h] = own * WIN + oct * (8 * PITCH + 16) + q * 8;
    }
    uint4 wreg[NT][4];
    const auto fetch = [&](int item, int q) {
        const int ts = item / a.slots, slot = item - ts * a.slots, tile = ts * PT + own, ty = tile / a.xtiles;
        const int iy0 = ty * RO * S - (N - 1) / 2, tx0 = (tile - ty * a.xtiles) * a.TW * S, ix0 = tx0 - (N - 1) / 2, o0 = (iy0 * a.W + ix0) * px2 + q * CK * 2;
        const int right = min(a.W, ix0 + (a.TW - 1) * S + N);         // columns that an output needs
        const __amdgpu_buffer_rsrc_t xr = __builtin_amdgcn_make_buffer_rsrc(
            (void*)(a.x + (int64_t)slot * a.H * a.W * a.C), 0, slot < a.B ? a.H * a.W * px2 : 0, 0x00020000);
#pragma unroll
        for (int h = 0; h < NT; ++h) {
            const bool ok = (unsigned)(prow[h] + iy0) < (unsigned)a.H && q * CK + oct * 8 < a.C;
            const int o = poff[h] + o0, ix = pcol[h] + ix0;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const auto v = __builtin_amdgcn_raw_buffer_load_b128(
                    xr, ok && (unsigned)(ix + k) < (unsigned)right ? o + k * px2 : (int)BAND_OOB, 0, 0);
                wreg[h][k] = make_uint4(v[0], v[1], v[2], v[3]);
            }
        }
    };
    short4_t A[CHUNKS][N][band_steps(N, S)];
    if constexpr (HOLD) {
        __syncthreads();
#pragma unroll
        for (int q = 0; q < CHUNKS; ++q) band_operand<N, S>(A[q], flt + (q * 16 + b) * FP);
    }

    fetch(blockIdx.x, 0);
    for (int item = blockIdx.x; item < a.items; item += gridDim.x) {
        const int slot = item % a.slots, tile = item / a.slots * PT + own, ty = tile / a.xtiles;
        const int oy0 = ty * RO, ox0 = (tile - ty * a.xtiles) * a.TW;
        f32x4_t acc[NP][2][MF];
#pragma unroll
        for (int j = 0; j < NP; ++j)
#pragma unroll
            for (int h = 0; h < 2; ++h)
#pragma unroll
                for (int m = 0; m < MF; ++m) acc[j][h][m] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int q = 0; q < CHUNKS; ++q) {
#pragma unroll
            for (int h = 0; h < NT; ++h) {
                if (prow[h] < K::ROWS) band_store_quads(win + plds[h], PITCH, wreg[h]);
            }
            __syncthreads();
            if (q + 1 < CHUNKS) fetch(item, q + 1);
            else if (item + gridDim.x < a.items) fetch(item + gridDim.x, 0);
            {
                f32x4_t d[RO];
                uint2 o[RO];
                const char *f = flt + (q * 16 + b) * FP, *p = win + own * WIN + cl * PITCH + (cl >> 3) * 16 + st * S * 8;
                if constexpr (!HOLD) band_operand<N, S>(A[q], f);
                band_rows<N, S, RO>(d, A[q], p, NQ);
                const float chk = band_finish<RO>(o, d, sc[q], sh[q], true);
                const int x = st * 4 + (odd ? 2 : 0), octet = sub * 2 + (b >> 3), in8 = (b & 6) * 2;
                const auto put = [&] {
#pragma unroll
                    for (int y = 0; y < RO; ++y) {
                        const uint2 t = band_trade(o[y], odd);
                        *(uint32_t*)(ops + (y * 16 + x) * (CK * 2) + turn<CK>(octet, x) * 16 + in8) = t.x;
                        *(uint32_t*)(ops + (y * 16 + x + 1) * (CK * 2) + turn<CK>(octet, x + 1) * 16 + in8) = t.y;
                    }
                };
                put();
                if (__ballot(chk != 0.f)) {
                    if (chk != 0.f) band_exact<N, S, RO>(o, sc[q], sh[q], true, f, p, NQ);
                    put();
                }
            }
            __syncthreads();
#pragma unroll
            for (int k = 0; k < K::KS; ++k) {
                if (q * K::KS + k >= KT) break;
                bf16x8_t pf[MF];
#pragma unroll
                for (int m = 0; m < MF; ++m)
                    pf[m] = *(const bf16x8_t*)(ops + (m * 16 + (lane & 15)) * (CK * 2) + turn<CK>(k * 4 + kg, lane & 15) * 16);
#pragma unroll
                for (int m = 0; m < MF; ++m)
#pragma unroll
                    for (int j = 0; j < NP; ++j)
#pragma unroll
                        for (int h = 0; h < 2; ++h)
                            acc[j][h][m] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[j][q * K::KS + k][h], pf[m], acc[j][h][m], 0, 0, 0);
            }
        }
        if (slot >= a.B || tile >= a.tiles) continue;
        const int x = lane & 15;
        const __amdgpu_buffer_rsrc_t yr = __builtin_amdgcn_make_buffer_rsrc(
            (void*)(a.y + (int64_t)slot * a.Ho * a.Wo * a.F), 0, a.Ho * a.Wo * a.F * 2, 0x00020000);
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            const int n = (sub + WT * j) * 32 + kg * 8;
            const int o = n < a.F && x < a.TW && ox0 + x < a.Wo ? (ox0 + x) * a.F * 2 + n * 2 : (int)BAND_OOB;
#pragma unroll
            for (int m = 0; m < MF; ++m) {
                if (oy0 + m >= a.Ho) break;
                float v[8];
#pragma unroll
                for (int k = 0; k < 8; ++k) v[k] = fmaxf(acc[j][k >> 2][m][k & 3] * s[j][k] + t[j][k], 0.f);
                typedef __attribute__((ext_vector_type(4))) uint32_t u4;
                const u4 r = {f2bf2(v[0], v[1]), f2bf2(v[2], v[3]), f2bf2(v[4], v[5]), f2bf2(v[6], v[7])};
                __builtin_amdgcn_raw_buffer_store_b128(r, yr, o, (oy0 + m) * a.Wo * a.F * 2, 0);
            }
        }
    }
}

template <int N, int S, int NW, int PT, int KT, int NP>
int32_t launch(BandPwArgs& a, hipStream_t s) {
    using K = BandPw<N, S, NW, PT, KT, NP>;
    a.tsets = (a.tiles + PT - 1) / PT;
    // a sample's tiles on one die where that costs few empty slots
    a.slots = a.B >= 32 ? (a.B + 7) & ~7 : a.B;
    const int64_t items = (int64_t)a.tsets * a.slots;
    if (items > 0x3fffffff) return DS_EUNSUPPORTED;
    a.items = (int)items;
    // as many workgroups as run at once, less what would leave the last ones idle
    const int at_once = 256 * K::AT_ONCE, rounds = (a.items + at_once - 1) / at_once;
    const int grid = std::min(a.items, ((a.items + rounds - 1) / rounds + 7) & ~7);
    const int32_t rc = ds_reserve_lds((const void*)bandpw_kernel<N, S, NW, PT, KT, NP>, K::SMEM, "separable block");
    if (rc) return rc;
    ProfScope prof(DS_K_DWCONV, s);
    hipLaunchKernelGGL((bandpw_kernel<N, S, NW, PT, KT, NP>), dim3(grid), dim3(NW * 64), K::SMEM, s, a);
    DS_CHECK_LAUNCH("depthwise-separable block");
    return DS_OK;
}

template <int N>
int32_t dispatch(BandPwArgs& a, int stride, hipStream_t s) {
    if (stride == 2) {
        if (a.C <= 32 && a.F <= 64) return launch<N, 2, 4, 2, 1, 1>(a, s);
        if (a.C <= 64 && a.F <= 128) return launch<N, 2, 4, 1, 2, 1>(a, s);
        if constexpr (N == 3)
            if (a.C <= 128 && a.F <= 256) return launch<N, 2, 8, 1, 4, 1>(a, s);
        return DS_EUNSUPPORTED;
    }
    if (a.C <= 32 && a.F <= 64) return launch<N, 1, 4, 2, 1, 1>(a, s);
    if (a.C <= 64 && a.F <= 128) return launch<N, 1, 4, 1, 2, 1>(a, s);
    if (a.C <= 128 && a.F <= 128) return launch<N, 1, 4, 1, 4, 1>(a, s);
    if constexpr (N == 3)
        if (a.C <= 256 && a.F <= 256) return launch<N, 1, 8, 1, 8, 1>(a, s);
    return DS_EUNSUPPORTED;
}

}  // namespace

int32_t ds_launch_bandpw(const bf16_t* x, int32_t B, int32_t H, int32_t W, int32_t C, const bf16_t* wd, int32_t KS, int32_t taps,
                         int32_t stride, const float* sd, const float* hd, const bf16_t* wp, int32_t F, const float* sp,
                         const float* hp, bf16_t* y, hipStream_t s) {
    if (B <= 0) return DS_OK;
    if (stride != 1 && stride != 2) return DS_EUNSUPPORTED;
    const int Ho = (H - 1) / stride + 1, Wo = (W - 1) / stride + 1;
    if (C % 8 || F % 8 || C < 8 || taps > KS || (KS - taps) % 2 || Wo <= 8 || (int64_t)H * W * C * 2 >= 0x7fffffffLL ||
        (int64_t)Ho * Wo * F * 2 >= 0x7fffffffLL)
        return DS_EUNSUPPORTED;
    BandPwArgs a = {};
    a.x = x; a.y = y; a.wd = wd; a.wp = wp; a.sd = sd; a.hd = hd; a.sp = sp; a.hp = hp;
    a.KS = KS; a.C = C; a.F = F; a.H = H; a.W = W; a.Ho = Ho; a.Wo = Wo; a.B = B; a.kb = (C + 31) / 32 | 1;
    a.xtiles = (Wo + 15) / 16;
    a.TW = (Wo + a.xtiles - 1) / a.xtiles;
    const int rows = stride == 1 ? 7 : 4;
    a.tiles = a.xtiles * ((Ho + rows - 1) / rows);
    if (taps == 3) return dispatch<3>(a, stride, s);
    if (taps == 5) return dispatch<5>(a, stride, s);
    return DS_EUNSUPPORTED;
}
