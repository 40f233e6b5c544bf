// 2D parallel- and fan-beam forward projection (ray-driven, a few lanes per
// detector bin) and back-projection (voxel-driven, a few waves per 8 x 8 pixels),
// Sec. II.B.2.  The images of the 2D workloads (at most 512 x 512 FP32,
// 1 MiB) stay resident in L2, so both kernels read global memory directly.
#include "device_util.h"

namespace ph {
namespace {

// Pixel (ix, iy), zero outside the image: read at the clamped index and
// masked, so that the loads of several samples are issued together.
template <typename T>
__device__ __forceinline__ float pix(const T *img, int nx, int ny, int ix, int iy)
{
    const int cx = min(max(ix, 0), nx - 1), cy = min(max(iy, 0), ny - 1);
    const float v = load_f32(img + (size_t)cy * nx + cx);
    return cx == ix && cy == iy ? v : 0.0f;
}

constexpr int UNROLL2D = 4;   // samples (A) or views (B) per lane whose loads are in flight together

// Narrow [lo, hi] to the sample range inside the open interval (a, b) of
// index coordinates.
__device__ __forceinline__ bool krange(float p, float e, float a, float b, float &lo, float &hi)
{
    if (fabsf(e) < 1e-30f)
        return p > a && p < b;
    const float r = 1.0f / e, t1 = (a - p) * r, t2 = (b - p) * r;
    lo = fmaxf(lo, fminf(t1, t2));
    hi = fminf(hi, fmaxf(t1, t2));
    return true;
}

// S lanes share one ray (S a power of two, at most 64: the lanes of a ray lie
// in one wave); lane s takes samples k0 + s, k0 + s + S, ... and the partial
// sums meet in a fixed shuffle tree.  Small problems (few rays, long rays)
// then still fill the machine.
//
// A lane takes four samples at a time.  Where every sample of the wave's four
// has its 2 x 2 cell inside the image (all but a ray's ends), the cell is
// read as two pairs at 32-bit offsets from the image, without bounds checks:
// 17 vector operations and two loads a sample.  Elsewhere the four pixels
// are read at clamped indices and masked.  (Four conditional loads per
// sample, each in a branch of its own, took 0.60 ms for 512^2 and 360 fan
// views of 725 bins; this takes 0.32 ms, bound by the scattered loads, about
// 40 clocks per CU for each.)
template <typename T, bool FAN, int S>
__global__ void __launch_bounds__(256) fp2d_kernel(Geom2D g, const float2 *__restrict__ views,
                                                   const T *__restrict__ img, T *__restrict__ sino, int n_rays,
                                                   int blocks)
{
    const int b = (int)(blockIdx.x / (unsigned)blocks);
    const long t = (long)(blockIdx.x % (unsigned)blocks) * 256 + threadIdx.x;
    const int r = (int)(t / S);
    const int s = (int)(t % S);
    if (r >= n_rays)
        return;   // whole rays only: the S lanes of a ray leave together
    const int j = r % g.nu, k = r / g.nu;
    const T *im = img + (size_t)b * g.nx * g.ny, *im1 = im + g.nx;
    float X0, Y0, eX, eY;
    make_ray_2d<FAN>(g, views[k], j, X0, Y0, eX, eY);
    float lo = -3.0e38f, hi = 3.0e38f;
    float acc = 0.0f;
    if (krange(X0, eX, -1.0f, (float)g.nx, lo, hi) && krange(Y0, eY, -1.0f, (float)g.ny, lo, hi) && lo < hi) {
        const int k0 = (int)floorf(lo) - 1, k1 = (int)ceilf(hi) + 1;
        // samples in_lo .. in_hi have their cells inside the image; the margin
        // covers the rounding of the clip and of the coordinates (relative 2^-22
        // of the anchor and of the image size), and 32-bit byte offsets must
        // reach the whole image
        const float ex = fmaf(1e-6f, (float)g.nx + fabsf(X0), 0.02f), ey = fmaf(1e-6f, (float)g.ny + fabsf(Y0), 0.02f);
        float ilo = -1.0e9f, ihi = 1.0e9f;
        const bool cells = krange(X0, eX, ex, (float)(g.nx - 1) - ex, ilo, ihi) &&
                           krange(Y0, eY, ey, (float)(g.ny - 1) - ey, ilo, ihi) &&
                           (size_t)g.nx * g.ny * sizeof(T) <= 0xffffffffu && g.nx < (1 << 24) && g.ny < (1 << 24);
        const int in_lo = cells ? (int)ceilf(ilo) : 1, in_hi = cells ? (int)floorf(ihi) : 0;
        for (int m = k0 + s; m <= k1; m += UNROLL2D * S) {
            if (__all(m >= in_lo && m + (UNROLL2D - 1) * S <= in_hi)) {
                float2 p[UNROLL2D], q[UNROLL2D];
                float tx[UNROLL2D], ty[UNROLL2D];
#pragma unroll
                for (int u = 0; u < UNROLL2D; ++u) {
                    const float fm = (float)(m + u * S), X = fmaf(fm, eX, X0), Y = fmaf(fm, eY, Y0);
                    tx[u] = __builtin_amdgcn_fractf(X);
                    ty[u] = __builtin_amdgcn_fractf(Y);
                    const unsigned off = (__umul24((unsigned)Y, (unsigned)g.nx) + (unsigned)X) * (unsigned)sizeof(T);
                    p[u] = load_pair(im, off);
                    q[u] = load_pair(im1, off);
                }
#pragma unroll
                for (int u = 0; u < UNROLL2D; ++u) {
                    const float a0 = fmaf(tx[u], p[u].y - p[u].x, p[u].x), a1 = fmaf(tx[u], q[u].y - q[u].x, q[u].x);
                    acc += fmaf(ty[u], a1 - a0, a0);
                }
            } else {
#pragma unroll
                for (int u = 0; u < UNROLL2D; ++u) {
                    const float fm = (float)(m + u * S), X = fmaf(fm, eX, X0), Y = fmaf(fm, eY, Y0);
                    const float fx = floorf(X), fy = floorf(Y);
                    const int ix = (int)fx, iy = (int)fy;
                    const float tx = X - fx, ty = Y - fy;
                    const float p00 = pix(im, g.nx, g.ny, ix, iy), p01 = pix(im, g.nx, g.ny, ix + 1, iy);
                    const float p10 = pix(im, g.nx, g.ny, ix, iy + 1), p11 = pix(im, g.nx, g.ny, ix + 1, iy + 1);
                    const float a0 = fmaf(tx, p01 - p00, p00), a1 = fmaf(tx, p11 - p10, p10);
                    const float v = fmaf(ty, a1 - a0, a0);
                    acc += m + u * S <= k1 ? v : 0.0f;
                }
            }
        }
    }
#pragma unroll
    for (int o = S / 2; o >= 1; o >>= 1)
        acc += __shfl_xor(acc, o);
    if (s == 0)
        store_f32(sino + ((size_t)b * g.n_proj + k) * g.nu + j, g.step * acc);
}

// A wave owns a tile of 8 x 8 pixels and takes one view at a time, so the view
// is uniform and its 64 reads fall on a dozen neighbouring bins of one row.
// The W waves of a workgroup share a tile, wave w taking views w, w + W, ...,
// and meet in LDS in a fixed order.  Four views' loads are in flight together;
// where both bins of all four lie on the detector for the whole wave, each
// pair is one load, otherwise two masked ones.  (With the lanes of a wave on 4
// views of 16 pixels: 174 against 112 us for 8 x 256^2 and 360 parallel views.)
template <typename T, typename TI, bool FAN>
__global__ void __launch_bounds__(1024) bp2d_kernel(Geom2D g, const float2 *__restrict__ views,
                                                    const TI *__restrict__ sino, T *__restrict__ img, int ntx, int nty)
{
    extern __shared__ float part[];   // one entry per thread, for more than one wave
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int waves = blockDim.x >> 6;
    const unsigned tile = blockIdx.x;
    const int tx = (int)(tile % (unsigned)ntx), ty = (int)((tile / (unsigned)ntx) % (unsigned)nty);
    const int b = (int)(tile / ((unsigned)ntx * (unsigned)nty));
    const int ix = tx * 8 + (lane & 7), iy = ty * 8 + (lane >> 3);
    const TI *sb = sino + (size_t)b * g.n_proj * g.nu;
    const float x = fmaf((float)min(ix, g.nx - 1), g.sx, g.ox), y = fmaf((float)min(iy, g.ny - 1), g.sy, g.oy);
    float acc = 0.0f;
    for (int k0 = wave; k0 < g.n_proj; k0 += UNROLL2D * waves) {
        float fu[UNROLL2D], t[UNROLL2D], wt[UNROLL2D];
        bool inside = true;
#pragma unroll
        for (int u = 0; u < UNROLL2D; ++u) {
            const int k = min(k0 + u * waves, g.n_proj - 1);
            point2d<FAN>(g, views[k], x, y, fu[u], t[u], wt[u]);
            inside = inside && fu[u] >= 0.0f && fu[u] < (float)(g.nu - 1);
        }
        if (__all(inside) && k0 + (UNROLL2D - 1) * waves < g.n_proj) {
            float2 p[UNROLL2D];
#pragma unroll
            for (int u = 0; u < UNROLL2D; ++u)
                p[u] = load_pair(sb + (size_t)(k0 + u * waves) * g.nu, (unsigned)fu[u] * (unsigned)sizeof(TI));
#pragma unroll
            for (int u = 0; u < UNROLL2D; ++u)
                acc = fmaf(wt[u], fmaf(t[u], p[u].y - p[u].x, p[u].x), acc);
        } else {
#pragma unroll
            for (int u = 0; u < UNROLL2D; ++u) {
                const int k = k0 + u * waves, j = (int)fu[u];
                const TI *row = sb + (size_t)min(k, g.n_proj - 1) * g.nu;
                const int j0 = min(max(j, 0), g.nu - 1), j1 = min(max(j + 1, 0), g.nu - 1);
                float p0 = load_f32(row + j0), p1 = load_f32(row + j1);
                p0 = j0 == j ? p0 : 0.0f;
                p1 = j1 == j + 1 ? p1 : 0.0f;
                const float v = fmaf(t[u], p1 - p0, p0);
                acc = k < g.n_proj ? fmaf(wt[u], v, acc) : acc;
            }
        }
    }
    if (waves > 1) {
        part[threadIdx.x] = acc;
        __syncthreads();
        if (wave > 0)
            return;
        for (int w = 1; w < waves; ++w)
            acc += part[w * 64 + lane];
    }
    if (ix < g.nx && iy < g.ny)
        store_f32(img + ((size_t)b * g.ny + iy) * g.nx + ix, g.dbeta * acc);
}

// Lanes per ray: up to about 2^21 threads in all (512^2, 360 fan views of 725
// bins: 312, 318, 365, 414 and 700 us for 16, 8, 4, 2 and 1 lanes; more lanes
// read more of each cache line while it is there), but at least 32 samples of
// the image's diagonal each, or setting the rays up outweighs sampling them
// (256^2, 30 parallel views: 21 us at 64 lanes, 16 us at 16).
inline int lanes_per_ray(const Geom2D &g, long rays)
{
    const float wx = g.nx * g.sx, wy = g.ny * g.sy, samples = sqrtf(wx * wx + wy * wy) / g.step;
    int S = 1;
    while (S < 64 && rays * S * 2 <= (1L << 21) && 64.0f * (float)S <= samples)
        S *= 2;
    return S;
}

template <typename T, bool FAN, int S>
hipError_t fp2d_s(const Geom2D &g, const float2 *views, const void *img, void *sino, int batch, hipStream_t s)
{
    const long n_rays = (long)g.nu * g.n_proj, blocks = (n_rays * S + 255) / 256;   // of one item
    if (n_rays > 0x7fffffffL || blocks * batch > 0x7fffffffL)
        return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL((fp2d_kernel<T, FAN, S>), dim3((unsigned)(blocks * batch)), dim3(256), 0, s, g, views,
                       (const T *)img, (T *)sino, (int)n_rays, (int)blocks);
    return hipGetLastError();
}

template <typename T, bool FAN>
hipError_t fp2d_f(const Geom2D &g, const float2 *views, const void *img, void *sino, int batch, hipStream_t s)
{
    switch (lanes_per_ray(g, (long)g.nu * g.n_proj * batch)) {
    case 1: return fp2d_s<T, FAN, 1>(g, views, img, sino, batch, s);
    case 2: return fp2d_s<T, FAN, 2>(g, views, img, sino, batch, s);
    case 4: return fp2d_s<T, FAN, 4>(g, views, img, sino, batch, s);
    case 8: return fp2d_s<T, FAN, 8>(g, views, img, sino, batch, s);
    case 16: return fp2d_s<T, FAN, 16>(g, views, img, sino, batch, s);
    case 32: return fp2d_s<T, FAN, 32>(g, views, img, sino, batch, s);
    default: return fp2d_s<T, FAN, 64>(g, views, img, sino, batch, s);
    }
}

template <typename T>
hipError_t fp2d(bool fan, const Geom2D &g, const float2 *views, const void *img, void *sino, int batch, hipStream_t s)
{
    return fan ? fp2d_f<T, true>(g, views, img, sino, batch, s) : fp2d_f<T, false>(g, views, img, sino, batch, s);
}

template <typename T, typename TI, bool FAN>
hipError_t bp2d_f(const Geom2D &g, const float2 *views, const void *sino, void *img, int batch, hipStream_t s)
{
    const int ntx = (g.nx + 7) / 8, nty = (g.ny + 7) / 8;
    const long tiles = (long)ntx * nty * batch;
    if (tiles > 0x7fffffffL)
        return hipErrorInvalidConfiguration;
    // waves per tile: at least 64 per CU in all (512^2, 360 fan views with the
    // filter: 107, 89, 86 and 89 us for 16, 32, 64 and 128), four views each
    int waves = 1;
    while (waves < 16 && tiles * waves < 16384 && 8 * waves <= g.n_proj)
        waves *= 2;
    hipLaunchKernelGGL((bp2d_kernel<T, TI, FAN>), dim3((unsigned)tiles), dim3(64 * waves),
                       waves > 1 ? 64 * waves * sizeof(float) : 0, s, g, views, (const TI *)sino, (T *)img, ntx, nty);
    return hipGetLastError();
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
