// Internal declarations shared by the HIP translation units of libdsnet.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdio.h>

#include "dsnet.h"
#include "quotient.h"

typedef uint16_t bf16_t;  // raw bfloat16 bits

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8_t;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16_t;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4_t;

// n / d, n not negative
__device__ __forceinline__ int ds_quotient(int n, int d) { return quotient(n, d, __builtin_amdgcn_rcpf((float)d)); }

__device__ __forceinline__ int ds_quotient_uniform(int n, int d) { return __builtin_amdgcn_readfirstlane(ds_quotient(n, d)); }

__device__ __forceinline__ float bf2f(bf16_t v) { return __uint_as_float(((uint32_t)v) << 16); }

// round-to-nearest-even float -> bf16 through the hardware conversion (v_cvt_pk_bf16_f32)
__device__ __forceinline__ bf16_t f2bf(float f) {
    const __bf16 b = (__bf16)f;
    return __builtin_bit_cast(bf16_t, b);
}
typedef __attribute__((ext_vector_type(2))) float f32x2_t;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2_t;
// two floats -> packed bf16 pair (lo in bits 0..15)
__device__ __forceinline__ uint32_t f2bf2(float lo, float hi) {
    const f32x2_t v = {lo, hi};
    const bf16x2_t b = __builtin_convertvector(v, bf16x2_t);
    return __builtin_bit_cast(uint32_t, b);
}

// ---- error reporting --------------------------------------------------------
void ds_set_error(const char* fmt, ...);
#define DS_FAIL(code, ...)            \
    do {                              \
        ds_set_error(__VA_ARGS__);    \
        return (code);                \
    } while (0)
#define DS_CHECK_LAUNCH(what)                                                  \
    do {                                                                       \
        hipError_t e__ = hipGetLastError();                                    \
        if (e__ != hipSuccess) DS_FAIL(DS_EHIP, "%s: %s", what, hipGetErrorString(e__)); \
    } while (0)

// reserves `bytes` of dynamic LDS for a kernel: once per (device, kernel), safe to call from any thread
int32_t ds_reserve_lds(const void* kernel, int bytes, const char* what);

static inline bool ds_aligned16(const void* p) { return (((uintptr_t)p) & 15u) == 0; }
static inline size_t ds_align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// ---- group table passed by value to kernels ---------------------------------
struct GroupTable {
    int32_t T;
    int32_t k_in[DS_MAX_GROUPS];
    int32_t k_out[DS_MAX_GROUPS];
    int32_t row[DS_MAX_GROUPS];
};

// per-group spatial slice of a stored KS x KS filter (Section 3.2, Eq. 11-13): the taps k0 + i*l, i < n, per axis
// (centred k x k block, every l-th tap), applied at dilation l with `pad` zeros per side
struct SpatialTable {
    int32_t k0[DS_MAX_GROUPS];
    int32_t n[DS_MAX_GROUPS];
    int32_t l[DS_MAX_GROUPS];
    int32_t pad[DS_MAX_GROUPS];
};

// ---- grouped GEMM / implicit-GEMM convolution -------------------------------
#define DS_GEMM_BM 128

struct GemmArgs {
    // operands
    const bf16_t* A;       // activations
    const bf16_t* Wt;      // weights [N_full][KK][w_tap_stride] (w_ld elements per output row)
    void* C;               // output
    const bf16_t* R;       // residual (nullable), addressed like C unless r_sample_stride is set
    const float* scale;    // [rows][tab_ld] nullable (=1)
    const float* shift;    // [rows][tab_ld] nullable (=0)
    // addressing: element offset of (slot, local row p, col) =
    //   index[slot] * sample_stride + (p + row0) * ld + col ;  ld <= 0 -> group's own width
    const int32_t* a_index;  // slot -> sample (nullable = identity)
    const int32_t* c_index;
    int64_t a_sample_stride, c_sample_stride, r_sample_stride;
    int32_t a_ld, c_ld, r_ld;
    int32_t c_row0;          // output/residual row shift inside a sample
    int32_t r_use_index;     // 0: residual ignores c_index (broadcast table such as a position embedding)
    // weights
    int64_t w_ld, w_tap_stride, w_seg_stride, c_seg_stride;
    int32_t n_seg, tab_ld, tab_seg_stride;
    // geometry: rows of a sample are the Ho*Wo output pixels of a KxK convolution over HxW
    int32_t H, W, Ho, Wo, K, stride, pad, rows;
    int32_t Kw, stride_w;    // filter width and horizontal stride where they differ from K / stride (0 = the same)
    // schedule
    const int32_t* offsets;  // device [T+1] slots; nullable: one group of B samples
    const int4* mtiles;      // device [(group, first row inside group, first slot, rows of group)]; nullable: the kernels
                             // work the record out from the offsets (saves the launch that builds the list)
    const int32_t* n_mtiles; // device scalar
    int32_t act, out_f32;
    int32_t B;               // samples of the launch, at most (0: unknown)
    int32_t crowd;           // launches like this one that run side by side (ds_forward_parts); 0 or 1: this one alone
    int32_t ordered;         // 1: every sum in channel order, as the 128-row kernels take it, whatever the batch size
    GroupTable gt;
};

#ifdef __HIPCC__
// inclusive sum over the lanes of a wavefront, without LDS round trips: rows of 16 lanes, then the last lane of each to the rows behind it
__device__ __forceinline__ int ds_scan64(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);
    return v;
}
// Record of the bm-row tile mt, found in the group offsets by the 64 lanes of the calling wavefront side by side; groups
// from the last to the first, as the tile lists have them.  .x < 0: there is no such tile.
__device__ __forceinline__ int4 ds_tile_record_of(const int32_t* offsets, int T, int rows, int mt, int bm) {
    const int lane = (int)(threadIdx.x & 63), g = T - 1 - lane, at = g >= 0 ? g : 0;
    int o0 = offsets[at], o1 = offsets[at + 1];
    if (g < 0) o0 = o1 = 0;
    const int rg = (o1 - o0) * rows, n = (rg + bm - 1) / bm;
    const int upto = ds_scan64(n);
    const unsigned long long past = __ballot(upto > mt);
    if (past == 0) return make_int4(-1, 0, 0, 0);
    const int q = __builtin_ctzll(past);
    const int before = __builtin_amdgcn_readlane(upto - n, q);
    return make_int4(T - 1 - q, (mt - before) * bm, __builtin_amdgcn_readlane(o0, q), __builtin_amdgcn_readlane(rg, q));
}
// Kernel arguments that a launch needs ahead of its first load, in scalar registers from here on.  Left to itself the compiler
// reads an argument in the basic block that uses it, so the head of a kernel with branches is a chain of a dozen dependent
// scalar loads of cold cache lines; held together they are one round trip.
template <typename T>
__device__ __forceinline__ void ds_hold1(T& v) { asm volatile("" : "+s"(v)); }
// (a pointer stays known as one to global memory: behind the asm it would be a generic one and its accesses flat)
template <typename T>
__device__ __forceinline__ void ds_hold1(T*& p) {
    uint64_t v = (uint64_t)p;
    asm volatile("" : "+s"(v));
    p = (T*)(__attribute__((address_space(1))) T*)v;
}
template <typename... T>
__device__ __forceinline__ void ds_hold(T&... v) { (ds_hold1(v), ...); }
// The group table by lanes: lane g holds group g's entries, requested together and ahead of the tile record, so that the
// slice widths are at hand when the group is known instead of one more dependent read of the kernel arguments.
struct GroupLanes {
    int ki, ko, ro;
    __device__ __forceinline__ explicit GroupLanes(const GroupTable& gt) {
        const int g = (int)(threadIdx.x & 63);
        static_assert(DS_MAX_GROUPS <= 64, "a lane per group");
        ki = gt.k_in[g];
        ko = gt.k_out[g];
        ro = gt.row[g];
    }
    __device__ __forceinline__ int k_in(int g) const { return __builtin_amdgcn_readlane(ki, __builtin_amdgcn_readfirstlane(g)); }
    __device__ __forceinline__ int k_out(int g) const { return __builtin_amdgcn_readlane(ko, __builtin_amdgcn_readfirstlane(g)); }
    __device__ __forceinline__ int row(int g) const { return __builtin_amdgcn_readlane(ro, __builtin_amdgcn_readfirstlane(g)); }
};
// Where the records of 128-row tiles come from, read with the other arguments (ds_hold).
struct TileSource {
    const int4* mtiles;
    const int32_t *n_mtiles, *offsets;
    int T, B, rows;
    __device__ __forceinline__ explicit TileSource(const GemmArgs& a)
        : mtiles(a.mtiles), n_mtiles(a.n_mtiles), offsets(a.offsets), T(a.gt.T), B(a.B), rows(a.rows) {}
    __device__ __forceinline__ void hold() { ds_hold(mtiles, n_mtiles, offsets, T, B, rows); }
    // record of tile mt: read from the list, or worked out where there is none (no offsets either: one group of B samples in slot order)
    __device__ __forceinline__ int4 record(int mt) const {
        if (mtiles) {
            const int4 me = mtiles[mt];          // in bounds even beyond the live count; checked next
            const int n = *n_mtiles;
            int x = __builtin_amdgcn_readfirstlane(me.x);
            ds_hold(x);                          // asked for beside the count, not behind it
            return mt < n ? make_int4(x, me.y, me.z, me.w) : make_int4(-1, 0, 0, 0);
        }
        if (!offsets) return mt * DS_GEMM_BM < B * rows ? make_int4(0, mt * DS_GEMM_BM, 0, B * rows) : make_int4(-1, 0, 0, 0);
        return ds_tile_record_of(offsets, T, rows, mt, DS_GEMM_BM);
    }
};
__device__ __forceinline__ int4 ds_tile_record(const GemmArgs& a, int mt) { return TileSource(a).record(mt); }
#endif

size_t ds_mtile_capacity(int32_t B, int32_t rows, int32_t T);
// ds_sliced_linear; with_ws: a workspace is demanded
int32_t ds_sliced_linear_on(const char* who, const void* x, int64_t x_ld, const void* w, int64_t w_ld, int32_t N_full,
                            int32_t K_full, const float* bias, const ds_groups* g, int32_t B, int32_t rows, int32_t act,
                            const void* residual, int64_t r_ld, void* y, int32_t y_dtype, int64_t y_ld, const void* ws,
                            size_t ws_bytes, bool with_ws, hipStream_t s);
int32_t ds_launch_gemm(const GemmArgs& a, int32_t max_mtiles, int32_t max_kout, hipStream_t s);
// 1x1 / linear layers with input slices of at most 64 channels and several 64-column passes: one workgroup per 128 rows
// and all their columns; DS_EUNSUPPORTED otherwise
int32_t ds_launch_thin(const GemmArgs& a, int32_t max_mtiles, int32_t max_kout, hipStream_t s);
// a second 1x1 layer applied to the rows of a thin layer before they leave the workgroup (Section 3.2: the next
// bottleneck's first convolution reads exactly the rows the previous bottleneck's last convolution wrote)
struct ThinChain {
    const bf16_t* Wt;              // [N2_full][w_ld]; its input slice is the first layer's output slice
    const float *scale, *shift;    // [rows][tab_ld], row = the group's row of the first layer; nullable (1 / 0)
    bf16_t* C;                     // second output: c_index[slot] * c_sample_stride + p * c_ld + col
    int64_t w_ld, c_sample_stride;
    int32_t c_ld, tab_ld, act;     // c_ld <= 0: the group's own width
    int32_t k_out[DS_MAX_GROUPS];  // per group; <= 0: the group ends with the first layer
};
int32_t ds_launch_thin_chain(const GemmArgs& a, const ThinChain& ch, int32_t max_mtiles, int32_t max_kout, hipStream_t s);
// launches too small for 128-row tiles: short tiles and a reduction dealt to several wavefronts; DS_EUNSUPPORTED otherwise
int32_t ds_launch_gemm_small(const GemmArgs& a, int32_t max_mtiles, int32_t max_kout, hipStream_t s);
// two 1x1 layers of a few samples as one launch; neither reads what the other writes
int32_t ds_launch_gemm_small_pair(const GemmArgs& a, int32_t mtiles_a, int32_t kout_a, const GemmArgs& b, int32_t mtiles_b, int32_t kout_b,
                                  hipStream_t s);
// whether ds_launch_gemm_small runs this layer
bool ds_gemm_small_takes(const GemmArgs& a, int32_t max_mtiles, int32_t max_kout);
// both as one launch of the 128-row kernel; DS_EUNSUPPORTED where either layer alone would take another kernel or another tile
int32_t ds_launch_gemm_pair(const GemmArgs& a, int32_t mtiles_a, int32_t kout_a, const GemmArgs& b, int32_t mtiles_b, int32_t kout_b, hipStream_t s);
// 3x3 stride-1 padding-1 layers on maps up to 59 pixels wide; DS_EUNSUPPORTED for any other shape
int32_t ds_launch_conv3(const GemmArgs& a, int32_t max_mtiles, int32_t max_kout, hipStream_t s);
// the same and those of stride 2 on filters in operand order (channels: as stored), without residual; DS_EUNSUPPORTED for other shapes and where another kernel is faster
int32_t ds_launch_conv3_tiled(const GemmArgs& a, const bf16_t* tiles, int32_t channels, int32_t max_mtiles, int32_t max_kout, hipStream_t s);
// the rest of a bottleneck block behind its first 1x1 layer (stride 1, packed rows, slot order): 3x3 layer, last 1x1 layer with its
// shortcut, the next block's first 1x1 layer; every one with batch-norm and ReLU.  DS_EUNSUPPORTED for shapes it is not written for and
// launches too small for it
struct BneckArgs {
    const bf16_t *y1, *w2, *w3, *w1;     // input; filters [mid_full][3][3][mid_full], [][mid_full], next block's [][out_full] (nullable)
    const float *s2, *h2, *s3, *h3, *s1, *h1;   // tables [row][mid_full], [row][tab3], [row][mid_full]
    const bf16_t* shortcut;              // addressed like z, may be z; or
    const bf16_t *x, *wp;                // (x not null) the stage's input and the projection's filters [][x_full]
    const float *sp, *hp;                // its tables [row][tab3]
    const int32_t* x_index;              // slot -> block of x
    bf16_t *z, *y1_next;
    float* sums;                         // null, or (no next block, slots of whole pieces) sums of z over pieces of 64 rows of a slot [slot][piece][out_full]
    int64_t y1_ss, z_ss, x_ss;           // elements per slot (y1_next as y1)
    int32_t mid_full, out_full, x_full, tab3, H, W;
    const int4* mtiles;
    const int32_t* n_mtiles;
    int32_t crowd;                       // as in GemmArgs
    GroupTable gt;                       // k_in = mid slice, k_out = output slice
    int32_t kx[DS_MAX_GROUPS], next[DS_MAX_GROUPS];   // slice of x; slice of the next block's first layer (<= 0: none)
};
bool ds_bneck_runs(const BneckArgs& a, int32_t B, int32_t max_mtiles);
int32_t ds_launch_bneck(const BneckArgs& a, int32_t B, int32_t max_mtiles, hipStream_t s);
constexpr int DS_BNECK_SUM_ROWS = 64;    // rows of a slot in a piece of BneckArgs::sums

static inline const int4* ds_mtile_entries(const void* list) { return (const int4*)((const char*)list + 16); }
static inline const int32_t* ds_mtile_count(const void* list) { return (const int32_t*)list; }

// ---- routing agent ------------------------------------------------------------
constexpr int POOL_SPLIT_MAX = 8;   // most partial sums per (item, channel) the spatial pool leaves for its consumer
struct GateArgs {
    const void* x;            // feature maps; nullptr = route on logit_bias alone
    int32_t dtype, layout;
    int32_t B, C, HW;         // items, stored channels, pixels
    const int32_t* c_in;      // per item valid channels (nullable = C)
    const int32_t* x_index;   // item -> sample block in x (nullable = identity)
    int64_t x_sample_stride;
    int32_t x_ld;             // NHWC row stride; <= 0 -> the item's own channel count
    const float *w1, *b1, *w2, *b2;
    int32_t C_mlp, T;
    const float* logit_bias;        // [*, T] indexed by output row, nullable
    const int32_t* out_index;       // item -> output row (nullable = identity)
    const int32_t* route_override;  // indexed by output row, nullable
    float* logits;
    int32_t* route;
    float* partial;           // [B][splits][C] scratch
    int32_t splits;           // > 0: the map's partial sums are there already
};
// whether a gate of these sizes takes partial sums made by the launch that wrote its map
bool ds_gate_takes_sums(const GateArgs& a);
size_t ds_gate_partial_bytes(int32_t B, int32_t C);
// y[b][p][c] = x[b][p][c] * scale[b][c] on the valid channels (NHWC) / y[b][c][p] (NCHW); fp32 or bf16
int32_t ds_launch_channel_scale(const void* x, void* y, const float* scale, const int32_t* c_in, int32_t dtype,
                                int32_t layout, int32_t B, int32_t C, int32_t HW, hipStream_t s);
constexpr int DS_BUCKET_LISTS = 4;
struct BucketArgs {
    const int32_t* route;     // [B]
    const int32_t* lo;        // nullable: key = route * mul + lo
    int32_t mul, B, T;
    int32_t *perm, *inv_perm, *offsets, *slot_group;   // inv_perm, slot_group nullable
    const int32_t* inv_prev;  // with src_index: src_index[slot] = inv_prev ? inv_prev[sample] : sample
    int32_t* src_index;       // nullable
    // optional extras done by the same launch (T <= DS_MAX_GROUPS): slot_lut[slot] = lut[group of slot], up to four m-tile lists for the new offsets (count, then
    // from byte 16 on one record per tile, ds_mtile_capacity() at most; list_rows[i] rows per sample), and the routes once more:
    // copy_to[i * copy_stride + sample], i < copies.  (What every launch reads comes first, in two lines of the scalar cache.)
    int32_t* slot_lut;        // nullable
    int32_t n_lists, list_rows[DS_BUCKET_LISTS];
    void* lists[DS_BUCKET_LISTS];
    int32_t lut[DS_MAX_GROUPS];
    int32_t* copy_to;
    int32_t copies, copy_stride;
};
int32_t ds_launch_bucket_ex(const BucketArgs& a, hipStream_t s);
// bucket (one sample, T <= 64): made by the gate's last launch itself, its route field is not read
int32_t ds_launch_gate(const GateArgs& a, hipStream_t s, const BucketArgs* bucket = nullptr);
int32_t ds_launch_bucket(const int32_t* route, int32_t B, int32_t T, int32_t* perm, int32_t* inv_perm,
                         int32_t* offsets, int32_t* slot_group, hipStream_t s);

// ---- memory-bound layers ------------------------------------------------------
// Activations are [slot][pixel or token][channel]; a slot's block starts at
// index[slot] * sample_stride and its rows have stride ld (<= 0: the slot's own width).
struct ActView {
    void* p;
    const int32_t* index;
    int64_t sample_stride;
    int32_t ld;
};

int32_t ds_launch_expand_groups(const int32_t* offsets, int32_t T, int32_t* slot_group, hipStream_t s);
int32_t ds_launch_dwconv(ActView x, ActView y, const bf16_t* w, const float* scale, const float* shift,
                         int32_t tab_ld, const int32_t* slot_group, const GroupTable& gt, int32_t B, int32_t C,
                         int32_t H, int32_t W, int32_t stride, int32_t act, hipStream_t s);
// spatially sliced filter; y is packed [Ho_t][Wo_t][ld] per slot, the resolution following the group's padding
int32_t ds_launch_dwconv_spatial(ActView x, ActView y, const bf16_t* w, int32_t KS, const float* scale, const float* shift,
                                 int32_t tab_ld, const int32_t* slot_group, const GroupTable& gt, const SpatialTable& st,
                                 int32_t B, int32_t C, int32_t H, int32_t W, int32_t stride, int32_t act, hipStream_t s);
// the same without dilation at stride 1 or 2, on the matrix cores; DS_EUNSUPPORTED otherwise
int32_t ds_launch_dwband(ActView x, ActView y, const bf16_t* w, int32_t KS, const float* scale, const float* shift, int32_t tab_ld,
                         const int32_t* slot_group, const GroupTable& gt, const SpatialTable& st, int32_t B, int32_t C, int32_t H,
                         int32_t W, int32_t stride, int32_t act, hipStream_t s);
// depthwise (3 x 3 or 5 x 5, stride 1 or 2, padding (taps - 1) / 2) and pointwise layer of a separable block in front of the
// gate with their batch-norms and ReLUs as one kernel; wp in operand tiles.  DS_EUNSUPPORTED for shapes it is not written for
int32_t ds_launch_bandpw(const bf16_t* x, int32_t B, int32_t H, int32_t W, int32_t C, const bf16_t* wd, int32_t KS, int32_t taps,
                         int32_t stride, const float* sd, const float* hd, const bf16_t* wp, int32_t F, const float* sp,
                         const float* hp, bf16_t* y, hipStream_t s);
// depthwise (3 x 3, padding 1, stride 1 or 2) and pointwise layer of a block behind the gate with their split batch-norms and
// ReLUs as one kernel; gt: k_in, k_out, table row of a route; wp in operand tiles, y [slot][pixel][k_out].  DS_EUNSUPPORTED
// for maps wider than a tile and slices beyond what LDS holds
int32_t ds_launch_sepconv(ActView x, bf16_t* y, int64_t y_ss, const bf16_t* wd, const float* sd, const float* hd, int32_t C,
                          const bf16_t* wp, const float* sp, const float* hp, int32_t F, const int32_t* slot_group,
                          const GroupTable& gt, int32_t B, int32_t H, int32_t W, int32_t stride, hipStream_t s);
// 3x3 stride-2 stem, a separable block at stride 1 and one at stride 2 (taps x taps filters cropped from KS x KS ones) as one
// kernel; wp0, wp1 in operand tiles.  DS_EUNSUPPORTED for shapes it is not written for
struct FrontLayers {
    const bf16_t *ws, *wd0, *wp0, *wd1, *wp1;
    const float *ss, *hs, *sd0, *hd0, *sp0, *hp0, *sd1, *hd1, *sp1, *hp1;
    int32_t C0, C1, F, KS0, KS1, taps;
};
int32_t ds_launch_front(const bf16_t* img, int32_t B, int32_t H, int32_t W, const FrontLayers& l, bf16_t* y, hipStream_t s);
int32_t ds_launch_layernorm(ActView x, ActView y, const float* gamma, const float* beta, float eps,
                            const int32_t* slot_group, const GroupTable& gt, int32_t B, int32_t rows,
                            int32_t row0, int32_t n_rows, hipStream_t s);
int32_t ds_launch_stem(const bf16_t* img, const int32_t* index, bf16_t* y, const bf16_t* w, const float* scale,
                       const float* shift, int32_t B, int32_t H, int32_t W, int32_t K, int32_t stride,
                       int32_t pad, int32_t Cout, hipStream_t s);
// 3x3 depthwise + batch-norm + ReLU and 1x1 pointwise + batch-norm + ReLU of an unsliced block in one kernel
// (x [B][H][W][C] -> y [B][Ho][Wo][N]); DS_EUNSUPPORTED when the shape has no fused variant
int32_t ds_launch_dwpw(const bf16_t* x, int32_t B, int32_t H, int32_t W, int32_t C, int32_t stride, const bf16_t* wd,
                       const float* sd, const float* hd, const bf16_t* wp, int32_t w_ld, int32_t N, const float* sp,
                       const float* hp, bf16_t* y, hipStream_t s);
int32_t ds_launch_stem_mfma(const bf16_t* img, const int32_t* index, bf16_t* y, const bf16_t* w, const float* scale,
                            const float* shift, int32_t B, int32_t H, int32_t W, int32_t K, int32_t stride,
                            int32_t pad, int32_t Cout, hipStream_t s);
int32_t ds_launch_maxpool(const bf16_t* x, bf16_t* y, int32_t B, int32_t H, int32_t W, int32_t C, hipStream_t s);
// fused 7x7/2 stem (64 filters) + 3x3/2 max-pool; DS_EUNSUPPORTED for other shapes
int32_t ds_launch_stem_pool(const bf16_t* img, const int32_t* index, bf16_t* y, const bf16_t* w, const float* scale,
                            const float* shift, int32_t B, int32_t H, int32_t W, int32_t K, int32_t stride,
                            int32_t pad, int32_t Cout, hipStream_t s);
// classifier: logits[out_index[slot]][o] = sum_{c < slot_c[slot]} W[o][c] * v[c] + b[o]; v = spatial mean of x
// (HW > 0; partial needs ds_gate_partial_bytes(B, C)) or row 0 of the slot (HW == 0)
int32_t ds_launch_head(ActView x, int32_t HW, const bf16_t* w, int32_t w_ld, const float* bias, int32_t n_out,
                       const int32_t* slot_c, const int32_t* out_index, float* logits, float* partial, int32_t B,
                       int32_t C, hipStream_t s);
int32_t ds_launch_patchify(const bf16_t* img, const int32_t* index, bf16_t* patches, int32_t B, int32_t H,
                           int32_t W, int32_t P, hipStream_t s);
int32_t ds_launch_cls_rows(ActView x, const bf16_t* cls, const bf16_t* pos, const int32_t* slot_group,
                           const GroupTable& gt, int32_t B, hipStream_t s);
int32_t ds_launch_conv_f32_nchw(const float* x, const float* w, const float* scale, const float* shift,
                                int32_t tab_ld, const float* residual, float* y, const int32_t* slot_group,
                                const int32_t* perm, const GroupTable& gt, int32_t B, int32_t C_I, int32_t C_O,
                                int32_t H, int32_t W, int32_t K, int32_t stride, int32_t pad, int32_t act,
                                hipStream_t s);
// 1x1 and 3x3 filters on the fp32 matrix cores, the slot's group read from the offsets; DS_EUNSUPPORTED otherwise
int32_t ds_launch_conv_f32_mfma(const float* x, const float* w, const float* scale, const float* shift, int32_t tab_ld,
                                const float* residual, float* y, const int32_t* offsets, const int32_t* perm,
                                const GroupTable& gt, int32_t B, int32_t C_I, int32_t C_O, int32_t H, int32_t W, int32_t K,
                                int32_t stride, int32_t pad, int32_t act, hipStream_t s);
int32_t ds_launch_lookup(const int32_t* idx, const GroupTable& gt, int32_t which, int32_t* out, int32_t B, hipStream_t s);

// ---- attention ----------------------------------------------------------------
// q, k, v, o: bf16 [slot][N][ld]; head j uses columns j*Dh..j*Dh+Dh-1; group g runs heads < k_out[g]/Dh;
// head_dim Dh: 32, 48 or 64
int32_t ds_launch_attention(const bf16_t* q, const bf16_t* k, const bf16_t* v, bf16_t* o, int64_t sample_stride,
                            int32_t ld, int32_t o_ld, int64_t o_sample_stride, const int32_t* slot_group,
                            const GroupTable& gt, int32_t B, int32_t N, int32_t H, int32_t head_dim, int32_t crowd, hipStream_t s);

// everything of a transformer block behind its attention.  Weights in operand order: [ceil(N / 32)][kb] tiles of 1 KiB, element (half h, row r, i) of a tile = W[32 nb + r][16 kb + 8 h + i], zeros
// beyond the stored matrix
struct VitTailArgs {
    const bf16_t* o;                     // attention output [slot][rows][o_ld]
    int64_t o_ss, x_ss;                  // elements per slot
    int32_t o_ld, rows;
    bf16_t* x;                           // residual stream, in place, packed rows
    const bf16_t *wp, *w1, *w2;          // projection, fc1, fc2
    int32_t kbp, kb1, kb2;               // 16-channel tiles per 32-row block
    const float *bp, *b1, *b2, *g2, *be2;
    float eps;
    const int32_t* offsets;
    // the next block's Q/K/V of the same rows, LayerNorm in front, where a group runs it (bit g of next)
    unsigned long long next;
    const bf16_t* wq;
    const float *bq, *g1, *be1;
    int32_t kbq, segq, q_ld;             // tiles per 32-row block, 32-row blocks and biases per segment (q_ld also the outputs' row stride)
    bf16_t* qkv;
    int64_t q_ss, q_seg;                 // elements per slot, per segment
    int32_t crowd;                       // as in GemmArgs
    GroupTable gt;                       // k_in = heads * head_dim, k_out = embedding slice, row = hidden slice
};
// y = act(LN(x) W^T + b) + residual on tiled weights
struct VitLinearArgs {
    const bf16_t* x;
    int64_t x_ss, y_ss, y_seg;           // elements per slot, per output segment
    int32_t x_ld, y_ld, rows;            // <= 0: packed rows
    const float *gamma, *beta;           // LayerNorm of the rows (nullable)
    float eps;
    const bf16_t* w;
    int32_t kb, seg_blocks, n_seg;       // 16-channel tiles and 32-row blocks per segment as stored
    const float* bias;
    int32_t bias_seg, act;
    const bf16_t* res;                   // addressed like y, nullable; may be y
    bf16_t* y;
    const int32_t* offsets;
    int32_t crowd;                       // as in GemmArgs
    GroupTable gt;
};
// DS_EUNSUPPORTED beyond 416 input channels with a LayerNorm, 1664 without
int32_t ds_launch_vit_linear(const VitLinearArgs& a, int32_t B, hipStream_t s);
// whether the next block's Q/K/V is to ride along; gt as in VitTailArgs
bool ds_vit_tail_qkv(const GroupTable& gt, int32_t B, int32_t rows, int32_t crowd);
// DS_EUNSUPPORTED where a slice exceeds 416 channels (hidden: any) or its alignment
int32_t ds_launch_vit_tail(const VitTailArgs& a, int32_t B, hipStream_t s);
// the same in tiles of 64 rows, two workgroups a compute unit; width: the widest slice of either kind (ds_launch_vit_tail's choice)
int32_t ds_launch_vit_duo(const VitTailArgs& a, int64_t tiles, int width, hipStream_t s);

// ---- per-kernel timing with HIP events (off unless ds_profile_enable(1)) ---------
enum {
    DS_K_GEMM = 0,   // gemm_kernel on linear / 1x1 layers
    DS_K_GEMM_TAPS,  // gemm_kernel walking KxK taps (implicit-GEMM convolution)
    DS_K_ATTENTION,
    DS_K_DWCONV,     // depthwise layers, alone or with the pointwise layer behind them in one kernel
    DS_K_LAYERNORM,
    DS_K_STEM,
    DS_K_MAXPOOL,
    DS_K_HEAD,
    DS_K_GATE,
    DS_K_BUCKET,
    DS_K_MISC,
    DS_K_CONV3,      // conv3_kernel, conv3_tiled_kernel (3x3 layers with the input patch staged once), bneck_kernel (a bottleneck block behind its first layer)
    DS_K_THIN,       // thin_kernel (short reductions, one workgroup per row tile; with or without a chained second layer)
    DS_K_TAIL,       // vit_tail_kernel, vit_duo_kernel (projection, MLP and LayerNorms of a transformer block)
    DS_K_SMALL,      // gemm_small_kernel (launches of a few samples, any filter size)
    DS_K_VIT_LINEAR, // vit_linear_kernel (linear layers on tiled weights, with or without the LayerNorm)
    DS_K_COUNT
};
struct ProfScope {
    int rec;
    hipStream_t s;
    ProfScope(int kind, hipStream_t stream);
    ~ProfScope();
};

struct ProfPause {   // no launch made by this thread inside its scope is recorded (and no event is created)
    bool was;
    ProfPause();
    ~ProfPause();
};

// ---- small dense layer on one vector per item --------------------------------------
struct FcArgs {
    const float* v_partial;   // [items][splits][C] partial sums (scaled by v_scale), or
    const bf16_t* v_rows;     // one bf16 row per item at v_rows + item * v_row_stride
    int64_t v_row_stride;
    int32_t splits;
    float v_scale;
    const int32_t* c_item;    // valid input width per item (nullable = C)
    int32_t C;                // stored input width / stride of v_partial
    const void* w;            // [n_out][w_ld] fp32 or bf16
    int32_t w_ld;
    const float* bias;        // nullable
    int32_t n_out, relu;      // relu: 0 none, 1 ReLU, 2 one plus tanh (attention head of the gate)
    const int32_t* out_index; // item -> output row (nullable = identity)
    float* out;
    int32_t out_ld, items;
};
int32_t ds_launch_fc(const FcArgs& a, int32_t w_bf16, int32_t acc_f64, int32_t kind, hipStream_t s);
// spatial partial sums of NHWC/NCHW feature maps into a.partial [B][splits][C]; returns splits
int32_t ds_launch_pool(const GateArgs& a, int32_t kind, int32_t* splits_out, hipStream_t s);
