// ds_sliced_linear for callers that cannot allocate device memory.  The grouped kernels find their row tiles in the group
// offsets, so there is no scratch at all: no state is shared between calls.  The size limit is the one of the array that
// the tile list used to be kept in; it is part of the interface.
#include "common.h"

extern "C" int32_t ds_sliced_linear_noalloc(const void* x, int64_t x_ld, const void* w, int64_t w_ld, int32_t N_full,
                                            int32_t K_full, const float* bias, const ds_groups* g, int32_t B,
                                            int32_t rows, int32_t act, const void* residual, int64_t r_ld, void* y,
                                            int32_t y_dtype, int64_t y_ld, void* stream) {
    const char* who = "ds_sliced_linear_noalloc";
    if (B < 0 || rows < 0) DS_FAIL(DS_EINVAL, "%s: negative size", who);
    if (!g) DS_FAIL(DS_EINVAL, "%s: null groups", who);
    if (g->T < 1 || g->T > DS_MAX_GROUPS) DS_FAIL(DS_EINVAL, "%s: T=%d outside 1..%d", who, g->T, DS_MAX_GROUPS);
    if (ds_mtile_capacity(B, rows, g->T) > (size_t)DS_NOALLOC_MAX_TILES)
        DS_FAIL(DS_EWORKSPACE, "%s: B * rows = %lld makes %zu row tiles, more than the %d of a call without workspace (the size "
                "of its former built-in scratch; use ds_sliced_linear)",
                who, (long long)B * rows, ds_mtile_capacity(B, rows, g->T), DS_NOALLOC_MAX_TILES);
    ProfPause quiet;   // kernel timing would create events on first use
    return ds_sliced_linear_on(who, x, x_ld, w, w_ld, N_full, K_full, bias, g, B, rows, act, residual, r_ld, y, y_dtype, y_ld,
                               nullptr, 0, false, (hipStream_t)stream);
}
