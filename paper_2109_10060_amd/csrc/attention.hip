// Head-sliced self-attention (Section 3.4, Eq. 17): one workgroup per (slot, head),
// heads at or beyond the slot's head count exit at once.  Head dimension 32, 48 or 64
// (DS-ViT++ stores 8 heads of 48: its Q-K-V widths 192..384 in steps of 48 go with 4..8 heads),
// sequence length up to 224 (7 key tiles of 32).
//
// K and V of the head live in LDS.  One wavefront per 32-query tile (up to 7 per workgroup):
//   S^T[key][q] = K . Q^T   (v_mfma_f32_32x32x16_bf16; A = K rows from LDS, B = Q rows from global)
// so that one lane owns a fixed query column and half of its keys: the row
// maximum and sum of the softmax are in-lane reductions plus one exchange with
// lane^32.  The probabilities are rounded to bf16 in registers and fed straight back as the B
// operand of  O^T = V^T . P^T  (normalised by the row sum afterwards, in fp32); the key order an accumulator
// holds (runs of 4 keys) is reproduced on the V^T side with two 8-byte LDS reads,
// so no shuffle or LDS round trip of P is needed.  V stays in rows in LDS and is transposed on the way out (read_keys): scattered into V^T two
// bytes at a time, the staging was a third of a workgroup's life.
#include <type_traits>

#include "common.h"

namespace {

constexpr int NKT = 7, KEYS = NKT * 32;

// Four keys of one channel out of rows of V: a group of 16 lanes reads 4 rows x 16 channels, 8 bytes a lane (row l16 / 4, channels 4 (l16 % 4) ..),
// and lane i gets channel i of the four rows.
typedef short s16x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint2 read_keys(const bf16_t* p) {
    const s16x4_t v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4_t*)p);
    return __builtin_bit_cast(uint2, v);
}

// DH: head dimension, a multiple of 16.  The output tiles are 32 channels tall; the channels past DH are computed from whatever lies
// there and dropped (they are rows of the product's first operand, so nothing else depends on them).
template <int DH>
__global__ __launch_bounds__(448) __attribute__((amdgpu_waves_per_eu(4, 4))) void attention_kernel(const bf16_t* __restrict__ q, const bf16_t* __restrict__ k,
                                                        const bf16_t* __restrict__ v, bf16_t* __restrict__ o,
                                                        int64_t sample_stride, int ld, int o_ld,
                                                        int64_t o_sample_stride, const int32_t* slot_group,
                                                        const GroupTable gt, int N, float scale) {
    constexpr int K_LD = DH + 8, KK = DH / 16, DT = (DH + 31) / 32, CPR = DH / 8;
    constexpr int V_LD = DT * 32 + 16;        // the four rows of a group of lanes on different banks
    static_assert(DH % 16 == 0 && DH <= 64, "head dimension");
    __shared__ __attribute__((aligned(16))) bf16_t Ks[KEYS * K_LD];
    __shared__ __attribute__((aligned(16))) bf16_t Vs[KEYS * V_LD];
    const int slot = blockIdx.x, head = blockIdx.y;
    const int width = gt.k_out[threadIdx.x & 63];            // (a lane per group: beside the group's number, not behind it)
    const int g = slot_group ? slot_group[slot] : 0;
    if (head * DH >= __builtin_amdgcn_readlane(width, __builtin_amdgcn_readfirstlane(g))) return;
    const int tid = threadIdx.x;
    const int64_t base = (int64_t)slot * sample_stride + head * DH;

    // this lane's query row, fetched first so that its latency overlaps the staging of K and V
    const int wave = tid >> 6, lane = tid & 63, l32 = lane & 31, lhi = lane >> 5;
    const int qrow = wave * 32 + l32;
    bf16x8_t qf[KK];
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
        uint4 t = make_uint4(0, 0, 0, 0);
        if (qrow < N) t = *(const uint4*)(q + base + (int64_t)qrow * ld + kk * 16 + lhi * 8);
        qf[kk] = *(bf16x8_t*)&t;
    }

    const int nthreads = blockDim.x;          // one wavefront per 32-query tile
    // A lane's pieces of K and V, four at a time (all there are with seven wavefronts of a 64-wide head), without a branch around a
    // request: rows past the sequence are past the descriptor and give zeros.  That is what lets them travel together; one at a time
    // measures the same (us a pass, four and one: 64 / 256 images of DS-ViT 892 / 2293 and 889 / 2289, 256 images of DS-ViT++ 3631 and 3639).
    constexpr int AT = 4;
    const int bytes = ((N - 1) * ld + DH) * 2;
    const __amdgpu_buffer_rsrc_t rk = __builtin_amdgcn_make_buffer_rsrc((void*)(k + base), 0, bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rv = __builtin_amdgcn_make_buffer_rsrc((void*)(v + base), 0, bytes, 0x00020000);
    for (int c0 = tid; c0 < KEYS * CPR; c0 += AT * nthreads) {
        uint4 kv[AT], vv[AT];
#pragma unroll
        for (int i = 0; i < AT; ++i) {
            const int c = c0 + i * nthreads, row = c / CPR, off = (row * ld + (c - row * CPR) * 8) * 2;
            const auto tk = __builtin_amdgcn_raw_buffer_load_b128(rk, off, 0, 0), tv = __builtin_amdgcn_raw_buffer_load_b128(rv, off, 0, 0);
            kv[i] = make_uint4(tk[0], tk[1], tk[2], tk[3]);
            vv[i] = make_uint4(tv[0], tv[1], tv[2], tv[3]);
        }
#pragma unroll
        for (int i = 0; i < AT; ++i) {
            const int c = c0 + i * nthreads, row = c / CPR, ch = (c - row * CPR) * 8;
            if (c >= KEYS * CPR) break;
            *(uint4*)(Ks + row * K_LD + ch) = kv[i];
            *(uint4*)(Vs + row * V_LD + ch) = vv[i];
        }
    }
    __syncthreads();
    // with few heads a workgroup multiplies for half of the query tiles only, one wavefront a SIMD
    if (gridDim.z > 1 && (wave >= 4) != (blockIdx.z > 0)) return;

    {
        // The keys are taken in two parts (tiles 0..3, then 4..6) with a running maximum and sum, so that only four
        // score tiles are alive at a time: 110 registers instead of 160, which lets two workgroups share a compute
        // unit and one of them stage its K and V while the other multiplies.  p = 2^((s - max) * scale * log2(e)),
        // masked keys get -inf; the scale is positive, so the maximum is taken on the raw scores.  The part's
        // probabilities are rounded to bf16 (relative to the running maximum), multiplied into O^T, and when the
        // maximum rises the earlier sum and O^T are scaled by 2^((old - new) * scale * log2(e)).
        const float c2 = scale * 1.44269504088896340736f;
        float m = -INFINITY, sum = 0.f;
        f32x16_t oacc[DT];
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int e = 0; e < 16; ++e) oacc[dt][e] = 0.f;
        const int vrow = 4 * lhi + ((lane & 15) >> 2), vcol = (lane & 16) + 4 * (lane & 3);   // what this lane reads for its group
        int krow = l32;                           // first key row of this lane; re-derived after each part (below)
        auto part = [&](auto lo_c, auto hi_c) {
            constexpr int LO = decltype(lo_c)::value, HI = decltype(hi_c)::value, NP = HI - LO;
            f32x16_t sacc[NP];
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                const int kt = LO + i;
#pragma unroll
                for (int e = 0; e < 16; ++e) sacc[i][e] = 0.f;
#pragma unroll
                for (int kk = 0; kk < KK; ++kk) {
                    const bf16x8_t kf = *(const bf16x8_t*)(Ks + (kt * 32 + krow) * K_LD + kk * 16 + lhi * 8);
                    sacc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[kk], sacc[i], 0, 0, 0);
                }
            }
            __builtin_amdgcn_sched_barrier(0);   // keep the phases apart: interleaving them costs the registers this split saves
            float mp = -INFINITY;
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                const int kt = LO + i;
                if (kt * 32 + 32 > N) {           // only the tiles that reach past the sequence need the mask
#pragma unroll
                    for (int e = 0; e < 16; ++e) {
                        const int key = kt * 32 + 8 * (e >> 2) + 4 * lhi + (e & 3);
                        if (key >= N) sacc[i][e] = -INFINITY;
                    }
                }
#pragma unroll
                for (int e = 0; e < 16; ++e) mp = fmaxf(mp, sacc[i][e]);
            }
            mp = fmaxf(mp, __shfl_xor(mp, 32, 64));
            if (LO > 0) {
                // a part with every key masked (N <= 128) leaves the maximum where it was and adds zeros
                const float mn = fmaxf(m, mp);
                const float alpha = __builtin_amdgcn_exp2f((m - mn) * c2);
                sum *= alpha;
#pragma unroll
                for (int dt = 0; dt < DT; ++dt)
#pragma unroll
                    for (int e = 0; e < 16; ++e) oacc[dt][e] *= alpha;
                m = mn;
            } else {
                m = mp;                           // key 0 is never masked: finite
            }
            const float mc = m * c2;
            __builtin_amdgcn_sched_barrier(0);
            uint32_t pf[NP][8];
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                float pr[16];
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    pr[e] = __builtin_amdgcn_exp2f(fmaf(sacc[i][e], c2, -mc));   // argument <= 0; results below 2^-126 flush to 0
                    sum += pr[e];
                }
#pragma unroll
                for (int e = 0; e < 8; ++e) pf[i][e] = f2bf2(pr[2 * e], pr[2 * e + 1]);
                asm volatile("" : "+v"(sum));        // the additions stay here: deferred, they keep all 16 values alive
                __builtin_amdgcn_sched_barrier(0);   // tile by tile: 16 scores become 8 packed registers before the next tile starts
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                const int kt = LO + i;
#pragma unroll
                for (int half = 0; half < 2; ++half) {
                    union { uint32_t u[4]; bf16x8_t v; } pv;
#pragma unroll
                    for (int e = 0; e < 4; ++e) pv.u[e] = pf[i][4 * half + e];
#pragma unroll
                    for (int dt = 0; dt < DT; ++dt) {
                        const bf16_t* vp = Vs + (kt * 32 + 16 * half + vrow) * V_LD + dt * 32 + vcol;
                        union { uint2 h[2]; bf16x8_t v; } vf;
                        vf.h[0] = read_keys(vp);
                        vf.h[1] = read_keys(vp + 8 * V_LD);
                        oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf.v, pv.v, oacc[dt], 0, 0, 0);
                    }
                }
            }
        };
        part(std::integral_constant<int, 0>{}, std::integral_constant<int, 4>{});
        // the second part's score tiles must not be started while the first part's probabilities are alive: tie the
        // address of its K reads to the end of the first part's O^T accumulation
        asm volatile("" : "+v"(krow) : "v"(oacc[0][0]), "v"(oacc[DT - 1][15]));
        part(std::integral_constant<int, 4>{}, std::integral_constant<int, NKT>{});
        sum += __shfl_xor(sum, 32, 64);
        const float inv = 1.0f / sum;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int e = 0; e < 16; ++e) oacc[dt][e] *= inv;
        // oacc[dt][e] = O[q = l32][d = dt*32 + 8*(e>>2) + 4*lhi + (e&3)]: the halves of the wavefront trade runs of 4 channels, so that
        // a lane stores 8 of them
        bf16_t* op = o + (int64_t)slot * o_sample_stride + (int64_t)qrow * o_ld + head * DH + 8 * lhi;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int g4 = 0; g4 < 4; g4 += 2) {
                if (dt * 32 + 8 * g4 >= DH) continue;   // padding channels of the last tile
                const uint32_t lo0 = f2bf2(oacc[dt][4 * g4], oacc[dt][4 * g4 + 1]), hi0 = f2bf2(oacc[dt][4 * g4 + 2], oacc[dt][4 * g4 + 3]);
                const uint32_t lo1 = f2bf2(oacc[dt][4 * g4 + 4], oacc[dt][4 * g4 + 5]), hi1 = f2bf2(oacc[dt][4 * g4 + 6], oacc[dt][4 * g4 + 7]);
                const auto a0 = __builtin_amdgcn_permlane32_swap(lo0, lo1, false, false);
                const auto a1 = __builtin_amdgcn_permlane32_swap(hi0, hi1, false, false);
                if (qrow < N) *(uint4*)(op + dt * 32 + 8 * g4) = make_uint4(a0[0], a1[0], a0[1], a1[1]);
            }
    }
}

}  // namespace

int32_t ds_launch_attention(const bf16_t* q, const bf16_t* k, const bf16_t* v, bf16_t* o, int64_t sample_stride,
                            int32_t ld, int32_t o_ld, int64_t o_sample_stride, const int32_t* slot_group,
                            const GroupTable& gt, int32_t B, int32_t N, int32_t H, int32_t head_dim, int32_t crowd, hipStream_t s) {
    if (B <= 0 || H <= 0) return DS_OK;
    if (N < 1 || N > KEYS) DS_FAIL(DS_EUNSUPPORTED, "attention: sequence length %d outside 1..%d", N, KEYS);
    if (head_dim != 32 && head_dim != 48 && head_dim != 64)
        DS_FAIL(DS_EUNSUPPORTED, "attention: head dimension %d (32, 48 or 64)", head_dim);
    ProfScope prof(DS_K_ATTENTION, s);
    const int waves = (N + 31) / 32;
    // Two workgroups a head, each with all keys and half of the query tiles, where that makes at most a workgroup a compute unit and the parts
    // of a batch that run side by side have no more heads than there are compute units.  Us a pass, one / two: DS-ViT, 20 images in two parts
    // (120 heads) 649 / 629, 32 in four (192) 726 / 714, 48 in four (288) 761 / 762, 64 in four (384) 869 / 900; DS-ViT++ 32 images in two (256) 1034
    // / 1022, 48 in four (384) 1118 / 1128
    const int64_t heads = (int64_t)B * H;
    const bool halves = waves > 4 && heads <= 128 && heads * (crowd > 1 ? crowd : 1) <= 256;
    const dim3 grid((unsigned)B, (unsigned)H, halves ? 2u : 1u), block(64 * waves);
    const float scale = 1.0f / sqrtf((float)head_dim);
#define DS_ATT(D)                                                                                                  \
    hipLaunchKernelGGL(attention_kernel<D>, grid, block, 0, s, q, k, v, o, sample_stride, ld, o_ld, o_sample_stride, \
                       slot_group, gt, N, scale)
    if (head_dim == 64) DS_ATT(64);
    else if (head_dim == 48) DS_ATT(48);
    else DS_ATT(32);
#undef DS_ATT
    DS_CHECK_LAUNCH("attention");
    return DS_OK;
}
