// What a tile of conv3_tiled_kernel keeps of its input in LDS, free of device types so that the host can check it.
#pragma once

#ifdef __HIP__
#define FIT_FN __host__ __device__ __forceinline__
#else
#define FIT_FN inline
#endif

// Pixels are counted with a column of zeros ahead of every map row and a row of zeros ahead of every sample, so that a tap is the same distance
// for every pixel and nothing is masked.  In LDS a pixel's 32 channels take CONV3_PITCH bytes and a map row begins CONV3_GAP bytes behind the last one's
// pixels (its zeros lie there, those of the column behind it too): neighbouring pixels of two map rows stay 80 bytes apart modulo the banks.
constexpr int CONV3_PITCH = 80, CONV3_GAP = 256;
constexpr int conv3_pixels(int bm) { return bm + 96; }                     // of a patch, at most
constexpr int conv3_bytes(int bm) { return bm == 128 ? 22784 : 17664; }    // of a patch

// whether the patch of any bm consecutive pixels of w x h maps fits; a tap reaches one padded row and one pixel beyond them
FIT_FN bool conv3_fits(int bm, int w, int h) {
    const int cross = (bm - 1) / w + 1, samples = (bm - 1) / (w * h) + 1;  // map rows, samples that bm pixels can end
    return bm + cross + samples * (w + 1) + 2 * (w + 2) <= conv3_pixels(bm) &&
           (cross + 1 + samples + 2) * (w * CONV3_PITCH + CONV3_GAP) <= conv3_bytes(bm);
}
// padded index of a pixel of a group
FIT_FN int conv3_padded(int sample, int y, int x, int w, int h) { return (sample * (h + 1) + y + 1) * (w + 1) + x + 1; }
// byte of padded index p in the patch whose first row is row0
FIT_FN int conv3_byte(int row, int col, int row0, int w) { return (row - row0) * (w * CONV3_PITCH + CONV3_GAP) + col * CONV3_PITCH; }

// Stride 2: output pixels are two input columns and two input rows apart.  Map rows are an even number of pixels apart, so that a tap is of one parity for
// every output pixel, and even and odd columns lie in planes of their own: neighbouring output pixels are neighbours there.
constexpr int CONV3_PIXELS2 = 488, CONV3_PLANE = CONV3_PIXELS2 / 2 * CONV3_PITCH, CONV3_BYTES2 = 2 * CONV3_PLANE;      // of a patch of 64 output pixels
FIT_FN int conv3_pitch2(int w) { return (w + 3) & ~1; }
// index of tap (0, 0) of an output pixel (even)
FIT_FN int conv3_padded2(int sample, int oy, int ox, int w, int h) { return (sample * (h + 1) + 2 * oy) * conv3_pitch2(w) + 2 * ox; }
FIT_FN bool conv3_fits2(int w, int h) {
    const int wo = (w - 1) / 2 + 1, ho = (h - 1) / 2 + 1, d = 63 / wo + 1, samples = 63 / (wo * ho) + 1, dx = 63 - wo * d;
    return (2 * d + samples * (h + 1 - 2 * ho) + 2) * conv3_pitch2(w) + 2 * dx + 3 <= CONV3_PIXELS2;
}
// byte of index p in the patch that begins with index first (even)
FIT_FN int conv3_byte2(int p, int first) { return (p & 1) * CONV3_PLANE + ((p - first) >> 1) * CONV3_PITCH; }
// bytes from tap (0, 0) to tap (u, v)
FIT_FN int conv3_tap2(int u, int v, int w) { return u * (conv3_pitch2(w) / 2) * CONV3_PITCH + (v == 1 ? CONV3_PLANE : v == 2 ? CONV3_PITCH : 0); }
