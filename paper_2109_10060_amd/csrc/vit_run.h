// Which columns of its output stage a workgroup of vit_linear_kernel owns, free of device types so that the host can check it.
#pragma once

#ifdef __HIP__
#define RUN_FN __host__ __device__ __forceinline__
#else
#define RUN_FN inline
#endif

// The stage holds nw column blocks from block b0 on as 16-byte chunks, four a block; a workgroup's run ends before block blk1.
// A chunk behind it is the next workgroup's: that one may be writing it, where residual and output are one buffer.
RUN_FN bool run_chunk(int c, int nw, int b0, int blk1) { return c < 4 * nw && b0 + (c >> 2) < blk1; }

// Segment of column block p of a layer of up to RUN_SEGMENTS stacked ones of nb blocks each.  (Two comparisons where p / nb, ahead of the first request
// and of every store, was a division.)
constexpr int RUN_SEGMENTS = 3;
RUN_FN int run_segment(int p, int nb) { return (p >= nb) + (p >= 2 * nb); }
