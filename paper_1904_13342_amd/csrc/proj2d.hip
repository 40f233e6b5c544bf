// 2D parallel- and fan-beam forward projection (ray-driven, one thread per
// detector bin) and back-projection (voxel-driven, one thread per pixel),
// Sec. II.B.2.  The images of the 2D workloads (at most 512 x 512 FP32,
// 1 MiB) stay resident in L2, so both kernels read global memory directly.
#include "device_util.h"

namespace ph {
namespace {

template <typename T>
__device__ __forceinline__ float pix(const T *img, int nx, int ny, int ix, int iy)
{
    return (ix >= 0 && iy >= 0 && ix < nx && iy < ny) ? load_f32(img + (size_t)iy * nx + ix) : 0.0f;
}

// Integer sample range covering the open box (-1, n) in index coordinates,
// widened by one sample on each side (samples outside add exact zeros).
__device__ __forceinline__ bool krange(float p, float e, int n, float &lo, float &hi)
{
    if (fabsf(e) < 1e-30f)
        return p > -1.0f && p < (float)n;
    float t1 = (-1.0f - p) / e, t2 = ((float)n - p) / e;
    lo = fmaxf(lo, fminf(t1, t2));
    hi = fminf(hi, fmaxf(t1, t2));
    return true;
}

// S lanes share one ray (S a power of two, at most 64: the lanes of a ray lie
// in one wave); lane s takes samples k0 + s, k0 + s + S, ... and the partial
// sums meet in a fixed shuffle tree.  Small problems (few rays, long rays)
// then still fill the machine.
template <typename T, bool FAN, int S>
__global__ void __launch_bounds__(256) fp2d_kernel(Geom2D g, const float2 *__restrict__ views,
                                                   const T *__restrict__ img, T *__restrict__ sino, long n_rays)
{
    const long t = (long)blockIdx.x * 256 + threadIdx.x;
    const long r = t / S;
    const int s = (int)(t % S);
    if (r >= n_rays)
        return;   // whole rays only: the S lanes of a ray leave together
    const int j = (int)(r % g.nu);
    const int k = (int)((r / g.nu) % g.n_proj);
    const int b = (int)(r / ((long)g.nu * g.n_proj));
    const T *im = img + (size_t)b * g.nx * g.ny;
    float X0, Y0, eX, eY;
    make_ray_2d<FAN>(g, views[k], j, X0, Y0, eX, eY);
    float lo = -3.0e38f, hi = 3.0e38f;
    float acc = 0.0f;
    if (krange(X0, eX, g.nx, lo, hi) && krange(Y0, eY, g.ny, lo, hi) && lo < hi) {
        const int k0 = (int)floorf(lo) - 1, k1 = (int)ceilf(hi) + 1;
#pragma unroll 4   // several samples' loads in flight at once
        for (int m = k0 + s; m <= k1; m += S) {
            const float fm = (float)m;
            const float X = fmaf(fm, eX, X0), Y = fmaf(fm, eY, Y0);
            const float fx = floorf(X), fy = floorf(Y);
            const int ix = (int)fx, iy = (int)fy;
            const float tx = X - fx, ty = Y - fy;
            const float p00 = pix(im, g.nx, g.ny, ix, iy), p01 = pix(im, g.nx, g.ny, ix + 1, iy);
            const float p10 = pix(im, g.nx, g.ny, ix, iy + 1), p11 = pix(im, g.nx, g.ny, ix + 1, iy + 1);
            const float a0 = fmaf(tx, p01 - p00, p00), a1 = fmaf(tx, p11 - p10, p10);
            acc += fmaf(ty, a1 - a0, a0);
        }
    }
#pragma unroll
    for (int o = S / 2; o >= 1; o >>= 1)
        acc += __shfl_xor(acc, o);
    if (s == 0)
        store_f32(sino + ((size_t)b * g.n_proj + k) * g.nu + j, g.step * acc);
}

template <typename T, typename TI, bool FAN, int S>
__global__ void __launch_bounds__(256) bp2d_kernel(Geom2D g, const float2 *__restrict__ views,
                                                   const TI *__restrict__ sino, T *__restrict__ img)
{
    // S lanes share a pixel of a 16 x (16 / S) block, 64 / S lanes apart, so
    // each run of 64 / S lanes reads adjacent pixels of one view; lane group s
    // takes views s, s + S, ... and the partial sums meet in a fixed shuffle
    // tree over the high lane bits
    constexpr int PW = 64 / S;   // pixels per wave
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int p = wave * PW + lane % PW, s = lane / PW;
    const int ix = blockIdx.x * 16 + (p & 15);
    const int iy = blockIdx.y * (16 / S) + (p >> 4);
    const int b = blockIdx.z;
    if (ix >= g.nx || iy >= g.ny)
        return;   // whole pixels only: the S lanes of a pixel leave together
    const TI *sb = sino + (size_t)b * g.n_proj * g.nu;
    const float x = fmaf((float)ix, g.sx, g.ox), y = fmaf((float)iy, g.sy, g.oy);
    float acc = 0.0f;
#pragma unroll 4   // several views' loads in flight at once
    for (int k = s; k < g.n_proj; k += S) {
        const float2 c = views[k];
        float fu, t, wt;
        point2d<FAN>(g, c, x, y, fu, t, wt);
        const int j = (int)fu;
        const TI *row = sb + (size_t)k * g.nu;
        const float p0 = (j >= 0 && j < g.nu) ? load_f32(row + j) : 0.0f;
        const float p1 = (j + 1 >= 0 && j + 1 < g.nu) ? load_f32(row + j + 1) : 0.0f;
        acc = fmaf(wt, fmaf(t, p1 - p0, p0), acc);
    }
#pragma unroll
    for (int o = 32; o >= PW; o >>= 1)
        acc += __shfl_xor(acc, o);
    if (s == 0)
        store_f32(img + ((size_t)b * g.ny + iy) * g.nx + ix, g.dbeta * acc);
}

// lanes per work item so that a launch holds about 2^21 threads (measured
// 20% faster than 2^20 for the 512^2 fan-beam sinogram, and ahead of 2^22)
inline int lanes_for(long items, int cap)
{
    int S = 1;
    while (S < cap && items * S * 2 <= (1L << 21))
        S *= 2;
    return S;
}

template <typename T, bool FAN, int S>
hipError_t fp2d_s(const Geom2D &g, const float2 *views, const void *img, void *sino, long n_rays, hipStream_t s)
{
    const long blocks = (n_rays * S + 255) / 256;
    hipLaunchKernelGGL((fp2d_kernel<T, FAN, S>), dim3((unsigned)blocks), dim3(256), 0, s, g, views, (const T *)img,
                       (T *)sino, n_rays);
    return hipGetLastError();
}

template <typename T, bool FAN>
hipError_t fp2d_f(const Geom2D &g, const float2 *views, const void *img, void *sino, long n_rays, hipStream_t s)
{
    switch (lanes_for(n_rays, 64)) {
    case 1: return fp2d_s<T, FAN, 1>(g, views, img, sino, n_rays, s);
    case 2: return fp2d_s<T, FAN, 2>(g, views, img, sino, n_rays, s);
    case 4: return fp2d_s<T, FAN, 4>(g, views, img, sino, n_rays, s);
    case 8: return fp2d_s<T, FAN, 8>(g, views, img, sino, n_rays, s);
    case 16: return fp2d_s<T, FAN, 16>(g, views, img, sino, n_rays, s);
    case 32: return fp2d_s<T, FAN, 32>(g, views, img, sino, n_rays, s);
    default: return fp2d_s<T, FAN, 64>(g, views, img, sino, n_rays, s);
    }
}

template <typename T>
hipError_t fp2d(bool fan, const Geom2D &g, const float2 *views, const void *img, void *sino, int batch, hipStream_t s)
{
    const long n_rays = (long)g.nu * g.n_proj * batch;
    return fan ? fp2d_f<T, true>(g, views, img, sino, n_rays, s) : fp2d_f<T, false>(g, views, img, sino, n_rays, s);
}

template <typename T, typename TI, bool FAN, int S>
hipError_t bp2d_s(const Geom2D &g, const float2 *views, const void *sino, void *img, int batch, hipStream_t s)
{
    dim3 grid((g.nx + 15) / 16, (g.ny + 16 / S - 1) / (16 / S), batch);
    hipLaunchKernelGGL((bp2d_kernel<T, TI, FAN, S>), grid, dim3(256), 0, s, g, views, (const TI *)sino, (T *)img);
    return hipGetLastError();
}

template <typename T, typename TI, bool FAN>
hipError_t bp2d_f(const Geom2D &g, const float2 *views, const void *sino, void *img, int batch, hipStream_t s)
{
    // lanes per pixel as for the projector's rays, at least two views per lane
    int cap = 16;
    while (cap > 1 && 2 * cap > g.n_proj)
        cap /= 2;
    switch (lanes_for((long)g.nx * g.ny * batch, cap)) {
    case 1: return bp2d_s<T, TI, FAN, 1>(g, views, sino, img, batch, s);
    case 2: return bp2d_s<T, TI, FAN, 2>(g, views, sino, img, batch, s);
    case 4: return bp2d_s<T, TI, FAN, 4>(g, views, sino, img, batch, s);
    case 8: return bp2d_s<T, TI, FAN, 8>(g, views, sino, img, batch, s);
    default: return bp2d_s<T, TI, FAN, 16>(g, views, sino, img, batch, s);
    }
}

template <typename T, typename TI>
hipError_t bp2d(bool fan, const Geom2D &g, const float2 *views, const void *sino, void *img, int batch,
                hipStream_t s)
{
    return fan ? bp2d_f<T, TI, true>(g, views, sino, img, batch, s) : bp2d_f<T, TI, false>(g, views, sino, img, batch, s);
}

}  // namespace

hipError_t launch_project_2d(int dtype, bool fan, const Geom2D &g, const float2 *views, const void *img, void *sino,
                             int batch, hipStream_t stream)
{
    switch (dtype) {
    case 0: return fp2d<float>(fan, g, views, img, sino, batch, stream);
    case 1: return fp2d<f16_t>(fan, g, views, img, sino, batch, stream);
    default: return fp2d<bf16_t>(fan, g, views, img, sino, batch, stream);
    }
}

hipError_t launch_backproject_2d(int dtype, bool fan, const Geom2D &g, const float2 *views, const void *sino,
                                 bool sino_is_f32, void *img, int batch, hipStream_t stream)
{
    switch (dtype) {
    case 0: return bp2d<float, float>(fan, g, views, sino, img, batch, stream);
    case 1:
        return sino_is_f32 ? bp2d<f16_t, float>(fan, g, views, sino, img, batch, stream)
                           : bp2d<f16_t, f16_t>(fan, g, views, sino, img, batch, stream);
    default:
        return sino_is_f32 ? bp2d<bf16_t, float>(fan, g, views, sino, img, batch, stream)
                           : bp2d<bf16_t, bf16_t>(fan, g, views, sino, img, batch, stream);
    }
}

}  // namespace ph
