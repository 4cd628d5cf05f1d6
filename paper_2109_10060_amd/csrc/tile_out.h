// What the kernels of 128-row tiles do with a finished tile.
#pragma once

#include "gelu.h"
#include <type_traits>

// LDS written and read by one wavefront: its accesses complete in order, only the compiler has to be kept in line
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
__device__ __forceinline__ void add_residual(float (&v)[4], const uint2 r) {
    v[0] += __uint_as_float(r.x << 16);
    v[1] += __uint_as_float(r.x & 0xffff0000u);
    v[2] += __uint_as_float(r.y << 16);
    v[3] += __uint_as_float(r.y & 0xffff0000u);
}
template <int ACT>
__device__ __forceinline__ void activate(float (&v)[4]) {
    if constexpr (ACT == DS_ACT_RELU) {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = fmaxf(v[e], 0.f);
    } else if constexpr (ACT == DS_ACT_GELU) {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = gelu_erf(v[e]);
    }
}
template <int ACT>
__device__ __forceinline__ uint2 activate_bf16(float (&v)[4]) {
    if constexpr (ACT == DS_ACT_GELU) return gelu_bf16x4(v[0], v[1], v[2], v[3]);
    activate<ACT>(v);
    return make_uint2(f2bf2(v[0], v[1]), f2bf2(v[2], v[3]));
}
// f with the activation as a constant; linear layers alone have GELU
template <bool LINEAR, class F>
__device__ __forceinline__ void with_act(int act, F&& f) {
    if (act == DS_ACT_RELU) return f(std::integral_constant<int, DS_ACT_RELU>());
    if constexpr (LINEAR) {
        if (act == DS_ACT_GELU) return f(std::integral_constant<int, DS_ACT_GELU>());
    }
    f(std::integral_constant<int, DS_ACT_NONE>());
}
inline bool conv_result(const GemmArgs& a) { return !a.out_f32 && a.act != DS_ACT_GELU; }
