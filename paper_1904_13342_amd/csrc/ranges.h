// Which samples of a ray to visit: host and device arithmetic in FP32, so that
// the bounds the kernels rely on can be checked on the CPU.
#pragma once

#include "common.h"

namespace ph {

// Narrow [lo, hi] to the sample range inside the open interval (a, b) of index
// coordinates; false where the ray never enters it, or it is empty.
__host__ __device__ __forceinline__ bool krange(float p, float e, float a, float b, float &lo, float &hi)
{
    if (!(a < b))
        return false;
    if (fabsf(e) < 1e-30f)
        return p > a && p < b;
    const float r = 1.0f / e, t1 = (a - p) * r, t2 = (b - p) * r;
    lo = fmaxf(lo, fminf(t1, t2));
    hi = fminf(hi, fmaxf(t1, t2));
    return true;
}

// Samples first .. last of the ray X0 + m eX, Y0 + m eY whose 2 x 2 cells lie
// inside the nx x ny image, so that they need no bounds checks; none (first >
// last) where that cannot be told.  The margin covers the rounding of the clip
// and of the coordinates (relative 2^-22 of the anchor and of the image size);
// an image of one row or column, or one that the margins use up, holds no cell.
// 32-bit byte offsets must reach the whole image.
__host__ __device__ __forceinline__ void cell_range(float X0, float Y0, float eX, float eY, int nx, int ny, size_t elem,
                                                    int &first, int &last)
{
    const float ex = fmaf(1e-6f, (float)nx + fabsf(X0), 0.02f), ey = fmaf(1e-6f, (float)ny + fabsf(Y0), 0.02f);
    float lo = -1.0e9f, hi = 1.0e9f;
    const bool cells = krange(X0, eX, ex, (float)(nx - 1) - ex, lo, hi) &&
                       krange(Y0, eY, ey, (float)(ny - 1) - ey, lo, hi) && lo <= hi &&
                       (size_t)nx * ny * elem <= 0xffffffffu && nx < (1 << 24) && ny < (1 << 24);
    first = cells ? (int)ceilf(lo) : 1;
    last = cells ? (int)floorf(hi) : 0;
}

// First guess at the sample after m, at coordinate at, that lies beyond bound,
// for rays that advance by 1 / rate; between m + 1 and last + 1 (compared as
// floats: a ray that hardly advances never gets there).  last - m < 2^24.
__host__ __device__ __forceinline__ int sample_beyond(int m, int last, float bound, float at, float rate)
{
    return m + (int)fmaxf(fminf(ceilf((bound - at) * rate), (float)(last + 1 - m)), 1.0f);
}

// How far beyond its clip (in steps) a ray is visited in the 3D A^T: 0.01 step,
// which covers the rounding of the clip, but at most half a voxel, so that no
// sample visited lies a voxel outside the box it was clipped to.  re_max = 1 /
// (largest increment of an index per step).
__host__ __device__ __forceinline__ float clip_margin(float re_max) { return fminf(0.01f, 0.5f * re_max); }

}  // namespace ph
