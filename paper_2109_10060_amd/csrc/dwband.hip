// Depthwise convolution with a spatially sliced filter (Section 3.2, Eq. 11 and 13: centred k x k block, k odd, no
// dilation) on the matrix cores.
//
// A filter row applied to four neighbouring outputs is a 4 x (N + 3) band matrix times a column of pixels, so one channel
// is one of the 16 blocks of v_mfma_f32_4x4x4_16b_bf16: operand A holds the band (zero off it), B four columns of pixels
// (four strips of the map), D four outputs of each.  Two or three steps of K = 4 do a filter row for 256 outputs at once,
// in 8 clocks each, where the vector units take 7 dot products (channels in pairs, as they lie) or 4 (taps in pairs) of 4
// clocks for every 64.
// A workgroup stages the input window of its TY x 4 TXS outputs for CW channels in LDS, channel by channel, and the filter
// with zeros around its rows.  A wavefront holds 16 channels' bands in registers and goes over 7 output rows of four strips
// at a time: every input row is read once and added to the (up to 7) output rows that it touches.  Maps are multiples of
// 7 high.
// Bound: memory at large batches (288..640 channels of 14x14, filters of 3 / 5 / 7 taps, 256 images: 34 us for 93 MB), a
// workgroup's chain of loads, LDS and stores at small ones (6 us for 8 images).  96 images: 17 us, against 28 us with dot
// products on channel pairs read straight from memory.
#include <algorithm>

#include "band.h"

namespace {

constexpr int RO = 7;          // output rows of a pass

struct BandArgs {
    ActView x, y;
    const bf16_t* w;
    const float *scale, *shift;
    const int32_t* slot_group;
    int32_t tab_ld, KS, C, H, W, act, B, slots8, TY, TXS, wbytes;   // TXS: strips of 4 outputs across a tile; wbytes: of the filter
    GroupTable gt;
    SpatialTable st;
};

template <int N, int STRIDE, int CW>
__device__ __forceinline__ void dwband_rows(const BandArgs& a, const char* win, const char* wts, int nq, int pitch, int strips,
                                          int slot, int g, int c, int cb, int oy0, int ox0, int Ho, int Wo) {
    constexpr int WH = 4 / (CW / 16);   // WH wavefronts per 16 channels
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int b = lane >> 2, cl = (wave / WH) * 16 + b, ch = cb * CW + cl;
    if (cb * CW + (wave / WH) * 16 >= c) return;
    short4_t A[N][band_steps(N, STRIDE)];
    const char* f = wts + cl * band_filter_pitch(N, STRIDE);
    band_operand<N, STRIDE>(A, f);
    const int64_t ti = (int64_t)a.gt.row[g] * a.tab_ld + min(ch, a.tab_ld - 1);
    const float sc = a.scale[ti], sh = a.shift[ti];
    const int ys = a.y.index ? a.y.index[slot] : slot, yld = a.y.ld > 0 ? a.y.ld : c;
    bf16_t* yb = (bf16_t*)a.y.p + (int64_t)ys * a.y.sample_stride + (ch & ~1);
    const bool odd = b & 1;
    const int n = odd ? 3 - (lane & 3) : lane & 3;              // strip; mirrored in odd channels, for the exchange below
    const int count = strips * (a.TY / RO);
    for (int u = wave % WH; u * 4 < count; u += WH) {
        const int sid = u * 4 + n, s1 = sid < count ? sid : 0;
        const int rc = s1 / strips, st = s1 - rc * strips;
        const char* p = win + cl * pitch + (cl >> 3) * 16 + (rc * RO * STRIDE * nq + st * STRIDE) * 8;
        f32x4_t acc[RO];
        band_rows<N, STRIDE, RO>(acc, A, p, nq);
        uint2 o[RO];
        const bool relu = a.act == DS_ACT_RELU;
        const float chk = band_finish<RO>(o, acc, sc, sh, relu);
        // a lane has 4 outputs of a channel; with its neighbour channel's lane it trades 2 of them, for 4-byte stores
        const int ox = ox0 + st * 4 + (odd ? 2 : 0), oy = oy0 + rc * RO;
        const auto put = [&] {
#pragma unroll
            for (int y = 0; y < RO; ++y) {
                const uint2 t = band_trade(o[y], odd);
                if (sid >= count || oy + y >= Ho || ch >= c) continue;
                bf16_t* yp = yb + (int64_t)((oy + y) * Wo + ox) * yld;
                if (ox < Wo) *(uint32_t*)yp = t.x;
                if (ox + 1 < Wo) *(uint32_t*)(yp + yld) = t.y;
            }
        };
        put();
        if (__ballot(chk != 0.f)) {
            if (chk != 0.f) band_exact<N, STRIDE, RO>(o, sc, sh, relu, f, p, nq);
            put();
        }
    }
}

// one-dimensional grid of (tiles x channel blocks) x (B rounded up to 8) slots, slot fastest: a sample stays on one die
template <int STRIDE, int CW>
__global__ __launch_bounds__(256) void dwband_kernel(const BandArgs a, const int cblocks, const int xtiles) {
    extern __shared__ __attribute__((aligned(16))) char smem[];   // filter [CW][N], window [CW][rows][quads] of 4 pixels
    const int slot = blockIdx.x % a.slots8, tid = threadIdx.x;
    if (slot >= a.B) return;
    for (int e = tid; e < a.wbytes / 16; e += 256) ((uint4*)smem)[e] = make_uint4(0, 0, 0, 0);   // zeros around the taps
    const int g = a.slot_group ? a.slot_group[slot] : 0;
    const int c = a.gt.k_in[g], n = a.st.n[g], pad = a.st.pad[g], k0 = a.st.k0[g];
    const int Ho = (a.H + 2 * pad - n) / STRIDE + 1, Wo = (a.W + 2 * pad - n) / STRIDE + 1;
    const int j = blockIdx.x / a.slots8, cb = j % cblocks, tile = j / cblocks;
    const int oy0 = tile / xtiles * a.TY, ox0 = tile % xtiles * a.TXS * 4;
    if (cb * CW >= c || oy0 >= Ho || ox0 >= Wo) return;
    const int strips = min(a.TXS, (Wo - ox0 + 3) / 4), nq = band_quads(strips, n, STRIDE);
    const int rows = (a.TY - 1) * STRIDE + n, pitch = band_pitch(rows, nq);
    char *wts = smem, *win = smem + a.wbytes;
    constexpr int CH8 = CW / 8;
    const int fp = band_filter_pitch(n, STRIDE);
    // the filter's taps: at most 49 x CH8 octets, one or two a lane
    constexpr int WL = (49 * CH8 + 255) / 256;
    uint4 wv[WL];
#pragma unroll
    for (int q = 0; q < WL; ++q) {
        const int e = min(tid + q * 256, n * n * CH8 - 1), t = e / CH8, i = t / n;
        wv[q] = *(const uint4*)(a.w + (int64_t)((k0 + i) * a.KS + k0 + t - i * n) * a.C + min(cb * CW + e % CH8 * 8, a.C - 8));
    }
    const int xs = a.x.index ? a.x.index[slot] : slot, xld = a.x.ld > 0 ? a.x.ld : c;
    const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
        (void*)((const bf16_t*)a.x.p + (int64_t)xs * a.x.sample_stride), 0, 0x7fffffff, 0x00020000);
    // four pixels of 8 channels -> 8 quads; zeros outside the image and past the slice
    const int total = rows * nq * CH8, inv = 65536 / nq + 1, ch = cb * CW + tid % CH8 * 8;
    const int iy0 = oy0 * STRIDE - pad, ix0 = ox0 * STRIDE - pad;
    char* wp = win + tid % CH8 * (8 * pitch + 16);
    __syncthreads();
    for (int e0 = tid; e0 < total; e0 += 512) {
        uint4 px[2][4];
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int q = (e0 + h * 256) / CH8, row = (q * inv) >> 16, ix = ix0 + (q - row * nq) * 4, iy = iy0 + row;
            const bool ok = iy >= 0 && iy < a.H && ch < c;
            const int o = ((iy * a.W + ix) * xld + ch) * 2;
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const auto t = __builtin_amdgcn_raw_buffer_load_b128(
                    rsrc, (int)(ok && ix + k >= 0 && ix + k < a.W ? (uint32_t)(o + k * xld * 2) : BAND_OOB), 0, 0);
                px[h][k] = make_uint4(t[0], t[1], t[2], t[3]);
            }
        }
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            if (h && e0 + 256 >= total) break;
            band_store_quads(wp + (e0 + h * 256) / CH8 * 8, pitch, px[h]);
        }
    }
#pragma unroll
    for (int q = 0; q < WL; ++q) {
        const int e = tid + q * 256, t = e / CH8, i = t / n;
        if (e < n * n * CH8) {
            bf16_t* p = (bf16_t*)(wts + e % CH8 * 8 * fp) + i * band_row_dwords(STRIDE) * 2 + band_lead(STRIDE) + t - i * n;
            const uint32_t* v = &wv[q].x;
#pragma unroll
            for (int k = 0; k < 8; ++k) p[k * (fp / 2)] = (bf16_t)(v[k / 2] >> (k & 1) * 16);
        }
    }
    __syncthreads();
    switch (n) {
        case 1: dwband_rows<1, STRIDE, CW>(a, win, wts, nq, pitch, strips, slot, g, c, cb, oy0, ox0, Ho, Wo); break;
        case 3: dwband_rows<3, STRIDE, CW>(a, win, wts, nq, pitch, strips, slot, g, c, cb, oy0, ox0, Ho, Wo); break;
        case 5: dwband_rows<5, STRIDE, CW>(a, win, wts, nq, pitch, strips, slot, g, c, cb, oy0, ox0, Ho, Wo); break;
        default: dwband_rows<7, STRIDE, CW>(a, win, wts, nq, pitch, strips, slot, g, c, cb, oy0, ox0, Ho, Wo); break;
    }
}

}  // namespace

int32_t ds_launch_dwband(ActView x, ActView y, const bf16_t* w, int32_t KS, const float* scale, const float* shift, int32_t tab_ld,
                         const int32_t* slot_group, const GroupTable& gt, const SpatialTable& st, int32_t B, int32_t C, int32_t H,
                         int32_t W, int32_t stride, int32_t act, hipStream_t s) {
    if (stride != 1 && stride != 2) return DS_EUNSUPPORTED;
    int nmax = 0, wo = 0, ho = 0, cmax = 0;
    for (int t = 0; t < gt.T; ++t) {
        const int n = st.n[t];
        if (st.l[t] != 1 || !(n & 1) || n > 7) return DS_EUNSUPPORTED;
        nmax = std::max(nmax, (int)n);
        ho = std::max(ho, (H + 2 * st.pad[t] - n) / stride + 1);
        wo = std::max(wo, (W + 2 * st.pad[t] - n) / stride + 1);
        cmax = std::max(cmax, (int)gt.k_in[t]);
    }
    if (B <= 0 || cmax <= 0 || ho <= 0 || wo <= 0) return DS_OK;
    // Tiles of at most 7 strips (28 outputs, or equal parts of a row) by 7 or 14 rows: three to five workgroups' windows
    // in a compute unit.  14 rows where that leaves 1024 workgroups and the window is under 48 KiB (288..640 channels of
    // 14x14, 256 images: 34 us, 43 in 7 rows; 96 images 17 and 21).  64 channels where 7 rows of 16 channels are one pass only
    // (maps up to 16 wide, at the smallest batches up to 8), so that every wavefront has one (800..1152 channels of 7x7, 256
    // images: 35 us, 39 with 32; 96 images 17 and 18; profiles/dispatch_choices.txt).
    const int sx = (wo + 3) / 4, xt = (sx + 6) / 7, txs = (sx + xt - 1) / xt;
    const auto bytes = [&](int cw, int ty) {
        return band_window(cw, band_pitch((ty - 1) * stride + nmax, band_quads(txs, nmax, stride))) + ((cw * band_filter_pitch(nmax, stride) + 15) & ~15);
    };
    const int slots8 = (B + 7) & ~7;
    int cw = 32, ty = RO;
    if (ho > RO && bytes(32, 2 * RO) <= 48 << 10 && (int64_t)((ho + 13) / 14) * xt * ((cmax + 31) / 32) * B >= 1024) ty = 2 * RO;
    if (txs * (ty / RO) <= (B < 32 ? 2 : 4) && cmax > 32 && bytes(64, ty) <= 64 << 10) cw = 64;
    const int cblocks = (cmax + cw - 1) / cw;
    const int64_t nwg = (int64_t)cblocks * xt * ((ho + ty - 1) / ty) * slots8;
    if (nwg > 0x7fffffffLL) return DS_EUNSUPPORTED;
    BandArgs a;
    a.x = x; a.y = y; a.w = w; a.scale = scale; a.shift = shift; a.slot_group = slot_group;
    a.tab_ld = tab_ld; a.KS = KS; a.C = C; a.H = H; a.W = W; a.act = act; a.B = B; a.slots8 = slots8; a.TY = ty; a.TXS = txs; a.wbytes = (cw * band_filter_pitch(nmax, stride) + 15) & ~15;
    a.gt = gt; a.st = st;
    ProfScope prof(DS_K_DWCONV, s);
    const int smem = bytes(cw, ty);
#define DS_BAND(S, CW)                                                                                                      \
    do {                                                                                                                    \
        const int32_t rc = ds_reserve_lds((const void*)dwband_kernel<S, CW>, 100 << 10, "depthwise bands");                 \
        if (rc) return rc;                                                                                                  \
        hipLaunchKernelGGL((dwband_kernel<S, CW>), dim3((unsigned)nwg), dim3(256), smem, s, a, cblocks, xt);                \
    } while (0)
    if (stride == 1 && cw == 32) DS_BAND(1, 32);
    else if (stride == 1) DS_BAND(1, 64);
    else if (cw == 32) DS_BAND(2, 32);
    else DS_BAND(2, 64);
#undef DS_BAND
    DS_CHECK_LAUNCH("spatial depthwise conv (bands)");
    return DS_OK;
}
