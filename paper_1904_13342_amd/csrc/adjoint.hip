// Exact transposes of the two operators (Sec. II.B.2 notes that the
// ray-driven projector and the voxel-driven back-projector are an unmatched
// pair; Eq. 4 and Sec. II.B.1 use A^T as A's gradient operator).
//
// A^T, the transpose of the fixed-step multilinear ray sampler: voxel j
// receives
//     step * sum_r g_r * sum_k Lambda(X_rk - j),
// Lambda the tensor-product hat function, X_rk the same FP32 sample positions
// the forward projector uses.  In 2D a thread owns a pixel and gathers, per
// view, over the rays that cross its support (j - 1, j + 1)^2, without
// atomics.  In 3D a workgroup owns a brick and its rays splat into an LDS
// accumulator (below).
//
// B^T in 2D, the transpose of the voxel-driven distance-weighted
// back-projector, gathers per detector bin over the pixels whose linear
// footprint covers it (FP32 output); the 3D B^T sits beside the back-projector
// it mirrors.
#include "device_util.h"
#include "ranges.h"

namespace ph {
namespace {

// --------------------------------------------------------------- A^T, 2D

// A wave owns a tile of 8 x 8 pixels, of up to eight items of a batch, and takes
// one view at a time.  The rays that can cross the tile (the bins of its
// footprint, a few dozen) are set up once for all its pixels, a ray per lane and
// up to four views at once, in double precision and exactly as the projector
// sets them up, and put in LDS with the reciprocals of their steps and their
// values; then every lane gathers over the two or three rays that cross its own
// pixel's support, clipping each to it.  Setting the ray up in every pixel
// instead is what the time went to: 3.19 ms for 512^2 and 360 fan views of 725
// bins, against 0.57 ms (0.80 ms setting up one view at a time); 256^2 with 30
// parallel views of 363 bins went from 46 to 15 us.  VALU-bound (1.06
// instructions a clock and CU at 512^2, 3% of them FP64), and the weights are the
// same for every item of a batch: another item costs one operation a ray.  Rays
// that are zero in every item add nothing: a wave passes over its chunk of views
// where all are (360 views of zeros, or of one value: 76 us).
// The W waves of a workgroup share a tile, wave w taking views w, w + W,
// ..., and meet in LDS in a fixed order.
template <int NB>
struct __align__(16) TileRay {
    float X0, Y0, eX, eY;   // sample m sits at (X0 + m eX, Y0 + m eY)
    float rX, rY;           // 1 / eX, 1 / eY (finite)
    float g[NB];            // the ray's value in each item
};

__device__ __forceinline__ float step_rcp(float e)
{
    // a ray that does not advance on this axis is inside the support on every
    // sample or on none
    return fabsf(e) < 1e-20f ? copysignf(1e20f, e) : __builtin_amdgcn_rcpf(e);
}

// max(1 - |d|, 0) in one instruction
__device__ __forceinline__ float hat(float d)
{
    float r;
    asm("v_sub_f32_e64 %0, 1.0, |%1| clamp" : "=v"(r) : "v"(d));
    return r;
}

//
// PX = 4: the wave's lanes hold a tile of 4 x 4 pixels four times over, each
// sixteen with one of the four views that are set up together, and add up at
// the end.  A small image then has four times the workgroups, of a quarter of
// the chain; it sets up two and a half times the rays for each pixel.
template <typename T, typename TI, bool FAN, int V, int NB, int PX>
__global__ void __launch_bounds__(1024) fpT2d_kernel(Geom2D g, const float2 *__restrict__ views,
                                                     const TI *__restrict__ sino, T *__restrict__ img, int ntx,
                                                     int nty, int batch, unsigned tile0)
{
    constexpr int L = 64 / V;   // lanes (and rays) per view
    static_assert(PX == 8 || (PX == 4 && V == 4), "a view to each group of pixels");
    extern __shared__ __align__(16) char at_lds[];   // 64 rays per wave
    TileRay<NB> *s_rays = (TileRay<NB> *)at_lds;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int waves = blockDim.x >> 6;
    TileRay<NB> *rays = s_rays + wave * 64;
    const unsigned tile = tile0 + blockIdx.x;
    const int tx = (int)(tile % (unsigned)ntx), ty = (int)((tile / (unsigned)ntx) % (unsigned)nty);
    const int b0 = NB * (int)(tile / ((unsigned)ntx * (unsigned)nty));
    const int ix = tx * PX + lane % PX, iy = ty * PX + lane / PX % PX;
    const float fx = (float)ix, fy = (float)iy;
    const float x = fmaf(fx, g.sx, g.ox), y = fmaf(fy, g.sy, g.oy);
    // this lane's corner of the tile's support (lane mod 4)
    const float qx = fmaf((float)((lane & 1) ? min(tx * PX + PX, g.nx) : tx * PX - 1), g.sx, g.ox);
    const float qy = fmaf((float)((lane & 2) ? min(ty * PX + PX, g.ny) : ty * PX - 1), g.sy, g.oy);
    const float margin = fmaf(1e-6f, (float)g.nu, 0.02f);   // rounding of the coordinates (bins)
    const size_t item = (size_t)g.n_proj * g.nu;
    float acc[NB];
#pragma unroll
    for (int n = 0; n < NB; ++n)
        acc[n] = 0.0f;
    for (int k0 = wave * V; k0 < g.n_proj; k0 += waves * V) {
        // the tile's bins in this lane's view
        const int kv = min(k0 + lane / L, g.n_proj - 1);
        const float2 cl = views[kv];
        int j_lo, j_hi;
        {
            float fu, t, wt;
            point2d<FAN, FORM_RANGE>(g, cl, qx, qy, fu, t, wt);
            const int jc = (int)fu;
            j_lo = max(imin4(jc), 0);
            j_hi = min(imax4(jc) + 1, g.nu - 1);
        }
        for (int c0 = 0; __any(j_lo + c0 <= j_hi); c0 += L) {
            const int jl = j_lo + c0 + lane % L;
            unsigned any = 0;   // a ray of zeros adds nothing
            if (jl <= j_hi) {
                TileRay<NB> r;
                make_ray_2d<FAN>(g, cl, jl, r.X0, r.Y0, r.eX, r.eY);
                r.rX = step_rcp(r.eX);
                r.rY = step_rcp(r.eY);
#pragma unroll
                for (int n = 0; n < NB; ++n) {
                    r.g[n] = load_f32(sino + min(b0 + n, batch - 1) * item + (size_t)kv * g.nu + jl);
                    any |= __float_as_uint(r.g[n]);
                }
                rays[lane] = r;
            }
            const unsigned long long some = __ballot(any != 0);
            if (some == 0)
                continue;
            wave_lds_fence();
            // the view's rays, in LDS from base + jv (bins jv .. je)
            auto gather = [&](float2 c, int jv, int je, int base) {
                // bins whose rays cross this pixel's support: its centre's
                // coordinate and a bound on the support's half width (central
                // projection of the box |dx| < sx, |dy| < sy; the fan angle
                // moves no faster than the slope)
                float fu, t, wt;
                point2d<FAN, FORM_RANGE>(g, c, x, y, fu, t, wt);
                const float ac = fabsf(c.x), as = fabsf(c.y);
                float h = fmaf(as, g.sx, ac * g.sy);
                if (FAN) {
                    const float xu = fmaf(y, c.x, -(x * c.y)), w = fmaf(x, c.x, fmaf(y, c.y, g.sid));
                    const float dw = fmaf(ac, g.sx, as * g.sy);
                    h = fmaf(fabsf(xu) * __builtin_amdgcn_rcpf(w), dw, h) * __builtin_amdgcn_rcpf(w - dw);
                }
                h = fmaf(h, g.ru, margin);
                const int ja = (int)ceilf(fmaxf(fu + (t - h), (float)jv)), jb = (int)floorf(fminf(fu + (t + h), (float)je));
                for (int j = ja; j <= jb; ++j) {
                    const TileRay<NB> r = rays[base + j];
                    // the samples inside the support; the clip only picks the
                    // range to visit (hardware reciprocals, widened), the
                    // weights decide every sample
                    const float cx = (fx - r.X0) * r.rX, cy = (fy - r.Y0) * r.rY;
                    const float lo = fmaxf(cx - fabsf(r.rX), cy - fabsf(r.rY));
                    const float hi = fminf(cx + fabsf(r.rX), cy + fabsf(r.rY));
                    if (!(lo < hi + 0.01f))
                        continue;
                    float w = 0.0f;
                    const int m1 = (int)floorf(hi + 0.02f);
                    for (int m = (int)ceilf(lo - 0.02f); m <= m1; ++m) {
                        const float wx = hat(fmaf((float)m, r.eX, r.X0) - fx);
                        const float wy = hat(fmaf((float)m, r.eY, r.Y0) - fy);
                        w = fmaf(wx, wy, w);
                    }
#pragma unroll
                    for (int n = 0; n < NB; ++n)
                        acc[n] = fmaf(r.g[n], w, acc[n]);
                }
            };
            if constexpr (PX == 8) {
#pragma unroll 1
                for (int v = 0; v < V && k0 + v < g.n_proj; ++v) {
                    const int jv = __builtin_amdgcn_readlane(j_lo, v * L) + c0;   // bin of the view's first ray
                    gather(views[k0 + v], jv, min(__builtin_amdgcn_readlane(j_hi, v * L), jv + L - 1), v * L - jv);
                }
            } else if (k0 + lane / L < g.n_proj) {
                gather(cl, j_lo + c0, min(j_hi, j_lo + c0 + L - 1), lane / L * L - j_lo - c0);
            }
            wave_lds_fence();
        }
    }
    if constexpr (PX == 4) {
#pragma unroll
        for (int n = 0; n < NB; ++n) {
            acc[n] += __shfl_xor(acc[n], 16);
            acc[n] += __shfl_xor(acc[n], 32);
        }
    }
    if (waves > 1) {
        __syncthreads();
        float *part = (float *)at_lds;
#pragma unroll
        for (int n = 0; n < NB; ++n)
            part[n * blockDim.x + threadIdx.x] = acc[n];
        __syncthreads();
        if (wave > 0)
            return;
        for (int w = 1; w < waves; ++w)
#pragma unroll
            for (int n = 0; n < NB; ++n)
                acc[n] += part[n * blockDim.x + w * 64 + lane];
    }
    if (ix < g.nx && iy < g.ny && lane < PX * PX)
#pragma unroll
        for (int n = 0; n < NB; ++n)
            if (b0 + n < batch)
                store_f32(img + ((size_t)(b0 + n) * g.ny + iy) * g.nx + ix, g.step * acc[n]);
}

// --------------------------------------------------------------- A^T, 3D
//
// A workgroup owns a 16 x 16 x 16 brick of voxels; each thread holds the
// FP64 sums of 8 voxels of it in registers, over every view.
// Per view, the rays that can reach the brick's support box (the detector
// pixels of its footprint: 8 corners projected by eight lanes and reduced with
// DPP) are set up exactly as the forward projector sets them up (FP64 set-up,
// the same biased FP32 sample positions, so the pair is transposed sample for
// sample) and clipped to the support box.  The rays are then counting-sorted
// by their number of samples, so the 64 rays a wave walks together have
// nearly equal lengths, and each lane walks one ray, splatting every sample's
// eight trilinear corner weights into an LDS accumulator.
//
// The accumulator holds 32-bit fixed-point integers (u32 LDS atomics issue
// in about half the time of FP64 ones, and integer sums are exact, so the
// result does not depend on the order of the adds).  The scale of a pass is
// set from its own rays: a sample's weight at one cell is at most 1, and the
// samples of one ray add at most 1 / e_max + 1 at a cell (e_max its largest
// per-step index increment), so no cell's sum exceeds
//     bound = sum over rays of |g_r| (1 / e_max,r + 1),
// and with scale = 2^30 / bound no cell can overflow.  Each corner term is
// rounded to the nearest integer; after the pass every thread adds its own
// cells, divided by the scale, to its FP64 sums and clears them.  The waves
// take the sorted rays in tasks of 64 from a shared counter, longest first.
//
// What the walk waits for is the LDS: rays of one length are mostly
// neighbours, and neighbours in step add to the same cells, which one atomic
// instruction serialises.  The lanes of a task therefore start an eighth of
// their rays apart and wrap round: at 256^3 (1.6 rays per voxel) address
// conflicts fell from 1.63e10 to 0.33e10 cycles and A^T of 248 views from
// 87 to 63 ms (2, 4, 8 and 16 starts, two of them walking backwards in the
// first: 73, 66, 63, 66 ms); at 512^3 (one ray per voxel) there were few and
// it gains 4%.  VALU and LDS are then busy 67 and 76% of the time.  512
// threads and a table of 1024 rays, so that a view's footprint is one pass (two
// workgroups fit a CU's LDS), measured 61 ms against 63 for 256 threads and 640
// rays (three workgroups), and 4.4 against 5.1 ms at 128^3; coarse detectors
// take the latter.
//
// Sample ranges come from a clip with hardware reciprocals (relative error
// ~1e-7 of a few thousand steps), widened by 0.01 step or half a voxel: every
// sample inside the support box is visited, and a visited sample lies less than
// a voxel outside it, so its cell is one of floor coordinates x0 - 2 .. x0 + 16
// and its corners reach x0 + 17.  Cells of the halo (x0 - 2, x0 - 1, x0 + 16 and
// x0 + 17 on any axis) are never read, since the neighbouring bricks own those
// voxels, so they need no clearing, and the first and the last share a column
// (of the row before), a row and a plane.  Rows and planes have odd pitches:
// even ones would put cells in line along an axis on a quarter of the banks.

constexpr int AT_B = 16;                       // brick edge (voxels)
constexpr int AT_PY = AT_B + 3;                // row pitch (words)
constexpr int AT_PZ = AT_PY * AT_PY;           // plane pitch (words)
constexpr int AT_ZERO = AT_PZ + AT_PY + 1;     // word of cell (x0 - 1, y0 - 1, z0 - 1)
constexpr int AT_CELLS = AT_ZERO + (AT_B + 3) * AT_PZ;
constexpr int AT_BINS = 256;                   // sample-count bins of the ray sort
constexpr float AT_FIX = 1073741824.0f;        // 2^30

template <typename T, typename TI, int AT_T, int AT_RAYS>
__global__ void __launch_bounds__(AT_T, AT_T == 512 ? 4 : 3) fpT_cone_kernel(
    Geom3D g, const ConeFPView *__restrict__ fviews, const ConeBPView *__restrict__ bviews,
    const TI *__restrict__ proj, T *__restrict__ vol, double *__restrict__ part, int nbx, int nby, int nbz,
    unsigned brick0)
{
    constexpr int AT_Z = AT_B * AT_B * AT_B / AT_T;   // voxels per thread (a piece of a z-column)
    constexpr int AT_PER_THREAD = (AT_RAYS + AT_T - 1) / AT_T;
    __shared__ int acc[AT_CELLS];
    __shared__ float4 s_ra[AT_RAYS];   // biased anchor X, Y, Z and the ray's value
    __shared__ float4 s_rb[AT_RAYS];   // step e_x, e_y, e_z and the first sample (int bits)
    __shared__ int s_cnt[AT_RAYS];
    __shared__ int hist[AT_BINS];
    __shared__ int s_wsum[AT_BINS / 64];
    __shared__ float s_wbound[AT_T / 64];
    __shared__ int s_nhit;
    __shared__ int s_next;   // next 64-ray task of the walk
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const unsigned brick = brick0 + blockIdx.x;
    const int bxi = (int)(brick % (unsigned)nbx), byi = (int)((brick / (unsigned)nbx) % (unsigned)nby);
    const int bzb = (int)(brick / (unsigned)(nbx * nby));
    const int bzi = bzb % nbz, b = bzb / nbz;
    const int x0 = bxi * AT_B, y0 = byi * AT_B, z0 = bzi * AT_B;
    for (int n = tid; n < AT_CELLS; n += AT_T)
        acc[n] = 0;
    if (tid < AT_BINS)
        hist[tid] = 0;
    if (tid == 0)
        s_next = 0;
    // this thread's voxels (x0 + lx, y0 + ly, z0 + lz .. z0 + lz + AT_Z - 1) and their cells
    const int lx = tid % AT_B, ly = (tid / AT_B) % AT_B, lz = tid / (AT_B * AT_B) * AT_Z;
    const int own = AT_ZERO + (lz + 1) * AT_PZ + (ly + 1) * AT_PY + lx + 1;   // cell of (lx, ly, lz); + AT_PZ per z
    double out[AT_Z];
#pragma unroll
    for (int z = 0; z < AT_Z; ++z)
        out[z] = 0.0;
    __syncthreads();

    const float hx = 0.5f * (g.nx - 1), hy = 0.5f * (g.ny - 1), hz = 0.5f * (g.nz - 1);
    // support box of the brick's voxels, (x0 - 1, min(x0 + B, N)) per axis:
    // inside the grid's support (-1, N), which the host has checked lies in
    // front of every source
    const int xe = min(x0 + AT_B, g.nx), ye = min(y0 + AT_B, g.ny), ze = min(z0 + AT_B, g.nz);
    // this lane's corner of the support box in centred voxel indices
    const int corner = tid & 7;
    const float bcx = (float)((corner & 1) ? xe : x0 - 1) - hx;
    const float bcy = (float)((corner & 2) ? ye : y0 - 1) - hy;
    const float bcz = (float)((corner & 4) ? ze : z0 - 1) - hz;
    // the same box in (unbiased) index coordinates, for the clip
    const float sx0 = (float)(x0 - 1), sx1 = (float)xe;
    const float sy0 = (float)(y0 - 1), sy1 = (float)ye;
    const float sz0 = (float)(z0 - 1), sz1 = (float)ze;
    // biased floor coordinate -> accumulator cell: floor(X) - (x0 - 1) = (int)(X + 4) - (x0 + 3);
    // the cell's byte address is 4 (iz PZ + iy PY + ix) + base (modulo 2^32)
    const unsigned base = 4u * (unsigned)AT_ZERO - 4u * (unsigned)((z0 + 3) * AT_PZ + (y0 + 3) * AT_PY + (x0 + 3));
    const TI *pb = proj + (size_t)b * g.n_proj * g.nv * g.nu;

    // this workgroup's share of the views
    const int k0 = (int)((long)g.n_proj * blockIdx.y / gridDim.y);
    const int k1 = (int)((long)g.n_proj * (blockIdx.y + 1) / gridDim.y);
    for (int k = k0; k < k1; ++k) {
        const ConeBPView bv = bviews[k];
        const float rw = rcp_nr(dot4(bv.r[2], bcx, bcy, bcz));
        const float cu = dot4(bv.r[0], bcx, bcy, bcz) * rw, cv = dot4(bv.r[1], bcx, bcy, bcz) * rw;
        // the corners' floors reduced as integers (floor is monotonic); the
        // sums are rounded on their own, not fused with the products above
        const int ju = (int)floorf(__fadd_rn(cu, g.cu)), iv = (int)floorf(__fadd_rn(cv, g.cv));
        const int j_lo = max(imin8(ju) - 1, 0), j_hi = min(imax8(ju) + 2, g.nu - 1);
        const int i_lo = max(imin8(iv) - 1, 0), i_hi = min(imax8(iv) + 2, g.nv - 1);
        const int W = j_hi - j_lo + 1, H = i_hi - i_lo + 1;
        if (W <= 0 || H <= 0)
            continue;
        const ConeFPView &fv = fviews[k];
        const TI *qk = pb + (size_t)k * g.nv * g.nu;
        const int nfp = W * H;
        const float rW = 1.0f / (float)W;
        for (int c0 = 0; c0 < nfp; c0 += AT_RAYS) {
            const int nc = min(AT_RAYS, nfp - c0);
            // set-up: this thread's footprint pixels of the pass
            float4 ra[AT_PER_THREAD], rb[AT_PER_THREAD];
            int cnt[AT_PER_THREAD];
            float lb = 0.0f;   // this thread's share of the bound
#pragma unroll
            for (int u = 0; u < AT_PER_THREAD; ++u) {
                cnt[u] = 0;
                const int idx = tid + AT_T * u;
                if (idx >= nc)
                    continue;
                // row and column of footprint pixel f (below 2^22 the rounded quotient is exact)
                const int f = c0 + idx, ii = nfp < (1 << 22) ? (int)(((float)f + 0.5f) * rW) : f / W;
                const int jj = f - ii * W;
                const int i = i_lo + ii, j = j_lo + jj;
                const float gv = load_f32(qk + (size_t)i * g.nu + j);
                if (gv == 0.0f)
                    continue;
                const Ray r = make_cone_ray(g, fv, j, i);
                const float re_max =
                    __builtin_amdgcn_rcpf(fmaxf(fabsf(r.e[0]), fmaxf(fabsf(r.e[1]), fabsf(r.e[2]))));
                const float eps = clip_margin(re_max);
                float lo = -3.0e38f, hi = 3.0e38f;
                if (!clip_line_rcp(r.p[0], r.e[0], sx0, sx1, lo, hi) ||
                    !clip_line_rcp(r.p[1], r.e[1], sy0, sy1, lo, hi) ||
                    !clip_line_rcp(r.p[2], r.e[2], sz0, sz1, lo, hi) || !(lo < hi + 2.0f * eps))
                    continue;
                const int m0 = (int)ceilf(lo - eps), m1 = (int)floorf(hi + eps);
                if (m1 < m0)
                    continue;
                cnt[u] = m1 - m0 + 1;
                ra[u] = make_float4(r.p[0] + RAY_BIAS, r.p[1] + RAY_BIAS, r.p[2] + RAY_BIAS, gv);
                rb[u] = make_float4(r.e[0], r.e[1], r.e[2], __int_as_float(m0));
                // 1 / e_max + 1, rounded up by a relative 1e-5 (the hardware reciprocal is within 1 ulp)
                lb = fmaf(fabsf(gv), fmaf(re_max, 1.00001f, 1.00001f), lb);
                atomicAdd(&hist[min(cnt[u], AT_BINS - 1)], 1);
            }
#pragma unroll
            for (int o = 32; o >= 1; o >>= 1)
                lb += __shfl_xor(lb, o);
            if (lane == 0)
                s_wbound[wave] = lb;
            __syncthreads();
            // slots in descending order of sample count: bin AT_BINS - 1 - tid
            // starts after the rays of all longer bins
            const int bin = AT_BINS - 1 - tid;
            int v = 0, x = 0;
            if (tid < AT_BINS) {   // whole waves
                v = x = hist[bin];
#pragma unroll
                for (int o = 1; o < 64; o <<= 1) {
                    const int y = __shfl_up(x, o);
                    if (lane >= o)
                        x += y;
                }
                if (lane == 63)
                    s_wsum[wave] = x;
            }
            __syncthreads();
            if (tid < AT_BINS) {
                int off = 0;
                for (int w = 0; w < wave; ++w)
                    off += s_wsum[w];
                hist[bin] = off + x - v;
                if (tid == AT_BINS - 1)
                    s_nhit = off + x;
            }
            __syncthreads();
#pragma unroll
            for (int u = 0; u < AT_PER_THREAD; ++u) {
                if (cnt[u] > 0) {
                    const int slot = atomicAdd(&hist[min(cnt[u], AT_BINS - 1)], 1);
                    s_ra[slot] = ra[u];
                    s_rb[slot] = rb[u];
                    s_cnt[slot] = cnt[u];
                }
            }
            __syncthreads();
            const int nhit = s_nhit;
            // summed in a fixed order: the result does not depend on the waves' timing
            float bound = 0.0f;
#pragma unroll
            for (int w = 0; w < AT_T / 64; ++w)
                bound += s_wbound[w];
            if (nhit > 0) {   // uniform
                const float scale = AT_FIX / bound;
                // the waves take 64-ray tasks in order of decreasing ray length
                for (;;) {
                    int t = 0;
                    if (lane == 0)
                        t = atomicAdd(&s_next, 1);
                    const int slot = __builtin_amdgcn_readfirstlane(t) * 64 + lane;
                    if (slot - lane >= nhit)
                        break;
                    if (slot >= nhit)
                        continue;
                    const float4 A = s_ra[slot], E = s_rb[slot];
                    const float gs = A.w * scale;
                    // every lane walks its whole ray, starting an eighth of it later than the
                    // lane before and wrapping round: neighbouring lanes hold neighbouring rays,
                    // which in step would add to the same cells
                    const int cnt_l = s_cnt[slot];
                    const float f0 = (float)__float_as_int(E.w), f1 = f0 + (float)cnt_l;
                    float fm = f0 + floorf((float)(lane & 7) * 0.125f * (float)cnt_l);
                    for (int n = cnt_l; n > 0; --n, fm = fm + 1.0f < f1 ? fm + 1.0f : f0) {
                        // the projector's biased sample position (positive: near the support box)
                        const float X = fmaf(fm, E.x, A.x), Y = fmaf(fm, E.y, A.y), Z = fmaf(fm, E.z, A.z);
                        const unsigned ix = (unsigned)X, iy = (unsigned)Y, iz = (unsigned)Z;
                        const float tx = __builtin_amdgcn_fractf(X), ty = __builtin_amdgcn_fractf(Y),
                                    tz = __builtin_amdgcn_fractf(Z);
                        unsigned off = 4u * (__umul24(iz, AT_PZ) + __umul24(iy, AT_PY) + ix) + base;
                        // the finished offset goes into one register, so the eight corners take
                        // immediate offsets (otherwise the constant part is split off per corner)
                        asm("" : "+v"(off));
                        int *c = (int *)((char *)acc + off);
                        const float a1 = gs * tz, a0 = gs - a1;
                        const float a01 = a0 * ty, a00 = a0 - a01, a11 = a1 * ty, a10 = a1 - a11;
                        // corner terms in fixed point, rounded to the nearest integer
                        atomicAdd(c, round_to_int(fmaf(-a00, tx, a00)));
                        atomicAdd(c + 1, round_to_int(a00 * tx));
                        atomicAdd(c + AT_PY, round_to_int(fmaf(-a01, tx, a01)));
                        atomicAdd(c + AT_PY + 1, round_to_int(a01 * tx));
                        atomicAdd(c + AT_PZ, round_to_int(fmaf(-a10, tx, a10)));
                        atomicAdd(c + AT_PZ + 1, round_to_int(a10 * tx));
                        atomicAdd(c + AT_PZ + AT_PY, round_to_int(fmaf(-a11, tx, a11)));
                        atomicAdd(c + AT_PZ + AT_PY + 1, round_to_int(a11 * tx));
                    }
                }
                __syncthreads();
                // fold this thread's cells into its FP64 sums and clear them
                const double inv = 1.0 / (double)scale;
#pragma unroll
                for (int z = 0; z < AT_Z; ++z) {
                    const int n = own + z * AT_PZ;
                    out[z] = fma((double)acc[n], inv, out[z]);
                    acc[n] = 0;
                }
            }
            if (tid < AT_BINS)
                hist[tid] = 0;
            if (tid == 0)
                s_next = 0;
            __syncthreads();
        }
    }
    if (part) {   // a share of the views: the brick's partial sums, thread by thread
        double *pp = part + ((size_t)blockIdx.y * gridDim.x + blockIdx.x) * (AT_B * AT_B * AT_B);
#pragma unroll
        for (int z = 0; z < AT_Z; ++z)
            pp[z * AT_T + tid] = out[z];
        return;
    }
    // write the brick's own voxels
    const size_t plane = (size_t)g.nx * g.ny;
    T *vb = vol + (size_t)b * g.nz * plane;
    const int ix = x0 + lx, iy = y0 + ly;
    if (ix < g.nx && iy < g.ny) {
#pragma unroll
        for (int z = 0; z < AT_Z; ++z)
            if (z0 + lz + z < g.nz)
                store_f32(vb + (size_t)(z0 + lz + z) * plane + (size_t)iy * g.nx + ix, (float)((double)g.step * out[z]));
    }
}

// Adds the shares' partial sums in order and writes the volume: one thread per
// voxel of a brick, in the order the bricks' threads wrote them.
template <typename T, int AT_T>
__global__ void __launch_bounds__(256) fpT_cone_sum_kernel(Geom3D g, const double *__restrict__ part,
                                                           T *__restrict__ vol, int nbx, int nby, int nbz, int shares,
                                                           unsigned bricks)
{
    constexpr int AT_Z = AT_B * AT_B * AT_B / AT_T;
    const unsigned brick = blockIdx.x / (AT_B * AT_B * AT_B / 256);
    const int e = (int)(blockIdx.x % (AT_B * AT_B * AT_B / 256)) * 256 + threadIdx.x;
    const int z = e / AT_T, t = e % AT_T;
    const int bxi = (int)(brick % (unsigned)nbx), byi = (int)((brick / (unsigned)nbx) % (unsigned)nby);
    const int bzb = (int)(brick / (unsigned)(nbx * nby));
    const int ix = bxi * AT_B + t % AT_B, iy = byi * AT_B + (t / AT_B) % AT_B;
    const int iz = bzb % nbz * AT_B + t / (AT_B * AT_B) * AT_Z + z;
    if (ix >= g.nx || iy >= g.ny || iz >= g.nz)
        return;
    const size_t stride = (size_t)bricks * (AT_B * AT_B * AT_B);
    const double *p = part + (size_t)brick * (AT_B * AT_B * AT_B) + e;
    double sum = 0.0;
    for (int s = 0; s < shares; ++s)
        sum += p[s * stride];
    store_f32(vol + (((size_t)(bzb / nbz) * g.nz + iz) * g.ny + iy) * g.nx + ix, (float)((double)g.step * sum));
}

// --------------------------------------------------------------- B^T, 2D

__global__ void fill_zero_kernel(float *__restrict__ p, size_t n)
{
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        p[i] = 0.0f;
}

// Gather over strips.  Strip j of a view holds the pixels whose detector
// coordinate su lies in [j, j + 1); each adds (1 - t) of its value to bin j
// and t to bin j + 1 (t = su - j).  A lane owns a strip and walks the image
// along the axis its strip crosses most slowly: one row (or column) of pixels
// at a time, the few candidates between the strip's two edge rays, each
// tested against the strip with the very coordinate the back-projector uses.
// Lane l then stores its own (1 - t) sum plus lane l - 1's t sum, so a wave
// of 64 strips writes 63 bins, every bin once: no atomics, no zero fill, and
// the same bits on every run.  The R waves of a workgroup share a wave's
// strips, each taking every R-th row, and meet in LDS.
//
// The scatter this replaces (two global float atomics per pixel and view,
// which neighbouring pixels aim at the same few bins) was bound by the
// atomics: 13.0 ms for 8 x 256^2 and 360 parallel views of 363 bins, against
// 0.48 ms (VALU-bound: about 100 lane operations per pixel and view).
struct StripEdge {
    float a, b;   // secondary index of the edge ray in row p of the walk: a + b p
};

// A point and the direction, in pixel indices, of the ray through detector
// coordinate u (bins) in a view with central ray c.
template <bool FAN>
__device__ __forceinline__ void edge_ray(const Geom2D &g, float2 c, double u, double &px, double &py, double &dx,
                                         double &dy)
{
    const double U = (u - (double)g.cu) * (double)g.du, cx = c.x, cy = c.y;
    if (!FAN) {
        px = -U * cy;
        py = U * cx;
        dx = cx;
        dy = cy;
    } else {
        px = -(double)g.sid * cx;
        py = -(double)g.sid * cy;
        double cg = (double)g.sdd, sg = U;
        if (g.curved)
            sincos(U / (double)g.sdd, &sg, &cg);
        dx = cg * cx - sg * cy;
        dy = cg * cy + sg * cx;
    }
    // index units
    px = (px - (double)g.ox) / (double)g.sx;
    py = (py - (double)g.oy) / (double)g.sy;
    dx /= (double)g.sx;
    dy /= (double)g.sy;
}

constexpr int STRIP_ROWS = 4;   // rows whose candidates are loaded together

// Called by whole waves; `used` is cleared for lanes without a strip.
template <typename TI, bool FAN, int AX, int FORM>
__device__ __forceinline__ void strip_walk(const Geom2D &g, float2 c, const TI *im, int j, bool used, bool bounded,
                                           StripEdge e0, StripEdge e1, int first, int stride, float &a0, float &a1)
{
    const int np = AX == 0 ? g.ny : g.nx, nq = AX == 0 ? g.nx : g.ny;
    // widest strip over the walk (pixels), and a margin for the rounding of
    // the edge lines and of the coordinates tested below
    const float w0 = fabsf(e1.a - e0.a), w1 = fabsf(fmaf(e1.b - e0.b, (float)(np - 1), e1.a - e0.a));
    const float wide = fmaxf(w0, w1), eps = fmaf(0.02f, wide, 0.02f);
    float lo = 0.0f, hi = (float)(np - 1);
    if (bounded) {
        // rows where the first edge is within a strip's width of the image
        const float qa = -1.0f - wide - eps, qb = (float)nq + wide + eps;
        if (fabsf(e0.b) > 1e-12f) {
            const float r = 1.0f / e0.b, t0 = (qa - e0.a) * r, t1 = (qb - e0.a) * r;
            lo = fmaxf(lo, fminf(t0, t1) - 1.0f);
            hi = fminf(hi, fmaxf(t0, t1) + 1.0f);
        } else if (!(e0.a > qa && e0.a < qb)) {
            hi = -1.0f;
        }
    }
    // rows and candidates per row are shared by the wave, so that its lanes
    // read neighbouring pixels of one row
    int p0 = (int)fminf(fmaxf(lo, 0.0f), (float)np), p1 = (int)fminf(fmaxf(hi, -1.0f), (float)(np - 1));
    int cand = bounded ? min((int)(wide + 2.0f * eps) + 1, nq) : nq;
    if (!used || p0 > p1) {
        p0 = np;
        p1 = -1;
        cand = 0;
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        p0 = min(p0, __shfl_xor(p0, o));
        p1 = max(p1, __shfl_xor(p1, o));
        cand = max(cand, __shfl_xor(cand, o));
    }
    p0 = __builtin_amdgcn_readfirstlane(p0);
    p1 = __builtin_amdgcn_readfirstlane(p1);
    cand = __builtin_amdgcn_readfirstlane(cand);
    const float jf = (float)j;
    p0 += (first - p0 % stride + stride) % stride;
    for (int pb = p0; pb <= p1; pb += STRIP_ROWS * stride) {
        int q0[STRIP_ROWS];
#pragma unroll
        for (int r = 0; r < STRIP_ROWS; ++r) {
            const float fp = (float)(pb + r * stride);
            const float qlo = bounded ? fminf(fmaf(fp, e0.b, e0.a), fmaf(fp, e1.b, e1.a)) - eps : 0.0f;
            q0[r] = (int)ceilf(fminf(fmaxf(qlo, 0.0f), (float)nq));
            if (pb + r * stride > p1)
                q0[r] = nq;   // past the last row: no candidates
        }
        for (int n = 0; n < cand; ++n) {
            float val[STRIP_ROWS];
#pragma unroll
            for (int r = 0; r < STRIP_ROWS; ++r) {
                const bool in = q0[r] + n < nq;
                const int q = in ? q0[r] + n : 0, p = in ? pb + r * stride : 0;
                val[r] = load_f32(im + (size_t)(AX == 0 ? p : q) * g.nx + (AX == 0 ? q : p));
            }
#pragma unroll
            for (int r = 0; r < STRIP_ROWS; ++r) {
                const bool in = q0[r] + n < nq;
                const int q = in ? q0[r] + n : 0, p = in ? pb + r * stride : 0;
                const int ix = AX == 0 ? q : p, iy = AX == 0 ? p : q;
                float fu, t, wt;
                point2d<FAN, FORM>(g, c, fmaf((float)ix, g.sx, g.ox), fmaf((float)iy, g.sy, g.oy), fu, t, wt);
                const float v = g.dbeta * wt * (in && fu == jf ? val[r] : 0.0f);
                a0 = fmaf(v, 1.0f - t, a0);
                a1 = fmaf(v, t, a1);
            }
        }
    }
}

template <typename TI, bool FAN>
__global__ void __launch_bounds__(1024) bpT2d_kernel(Geom2D g, const float2 *__restrict__ views,
                                                     const TI *__restrict__ img, float *__restrict__ sino, int groups,
                                                     unsigned block0)
{
    extern __shared__ float2 part[];   // one entry per thread, for more than one wave
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = blockDim.x >> 6;
    const unsigned block = block0 + blockIdx.x;
    const int grp = (int)(block % (unsigned)groups);
    const long kb = block / (unsigned)groups;   // view of an item
    const int k = (int)(kb % g.n_proj), b = (int)(kb / g.n_proj);
    const int j = grp * 63 - 1 + lane;   // this lane's strip
    const float2 c = views[k];
    const TI *im = img + (size_t)b * g.nx * g.ny;
    float a0 = 0.0f, a1 = 0.0f;
    {
        const bool used = j < g.nu;
        const double jd = (double)(used ? j : g.nu - 1);
        double px, py, dx0, dy0, qx, qy, dx1, dy1;
        edge_ray<FAN>(g, c, jd, px, py, dx0, dy0);
        edge_ray<FAN>(g, c, jd + 1.0, qx, qy, dx1, dy1);
        // the wave walks along the axis its first strip's edges advance on
        // faster (its strips span a few degrees); a strip whose edges do not
        // both advance one way along it (a bin wider than a right angle, say)
        // is not bounded by them: every pixel of a row is a candidate
        const int ax = __builtin_amdgcn_readfirstlane(fabs(dy0) + fabs(dy1) >= fabs(dx0) + fabs(dx1) ? 0 : 1);
        const double p0 = ax == 0 ? dy0 : dx0, p1 = ax == 0 ? dy1 : dx1;
        const double s0 = ax == 0 ? dx0 : dy0, s1 = ax == 0 ? dx1 : dy1;
        const bool bounded = p0 * p1 > 0.0 && fabs(p0) > 0.05 * fabs(s0) && fabs(p1) > 0.05 * fabs(s1);
        StripEdge e0 = {0.0f, 0.0f}, e1 = {0.0f, 0.0f};
        if (bounded) {
            const double b0 = s0 / p0, b1 = s1 / p1;
            e0.b = (float)b0;
            e1.b = (float)b1;
            e0.a = (float)(ax == 0 ? px - py * b0 : py - px * b0);
            e1.a = (float)(ax == 0 ? qx - qy * b1 : qy - qx * b1);
        }
        with_form<FAN>(g, [&](auto form) {
            if (ax == 0)
                strip_walk<TI, FAN, 0, decltype(form)::value>(g, c, im, j, used, bounded, e0, e1, wave, waves, a0, a1);
            else
                strip_walk<TI, FAN, 1, decltype(form)::value>(g, c, im, j, used, bounded, e0, e1, wave, waves, a0, a1);
        });
    }
    if (waves > 1) {
        part[threadIdx.x] = make_float2(a0, a1);
        __syncthreads();
        if (wave > 0)
            return;
        for (int w = 1; w < waves; ++w) {
            const float2 o = part[w * 64 + lane];
            a0 += o.x;
            a1 += o.y;
        }
    }
    const float below = __shfl_up(a1, 1);
    if (lane > 0 && j < g.nu)
        sino[((size_t)b * g.n_proj + k) * g.nu + j] = a0 + below;
}

// The value of the next or previous lane of the wave (DPP wavefront shifts by
// one), `end` in the last or first one.
__device__ __forceinline__ int next_lane(int x, int end)
{
    return __builtin_amdgcn_update_dpp(end, x, 0x130, 0xF, 0xF, false);
}
__device__ __forceinline__ float next_lane(float x, float end)
{
    return __int_as_float(next_lane(__float_as_int(x), __float_as_int(end)));
}
__device__ __forceinline__ int prev_lane(int x, int end)
{
    return __builtin_amdgcn_update_dpp(end, x, 0x138, 0xF, 0xF, false);
}

// The same gather from the pixels' side, where a view's bins fit a wave's LDS.
// A wave takes runs of 64 neighbouring pixels along the axis on which the
// detector coordinate moves faster, one run after the other, and adds each
// pixel's two terms to the (1 - t, t) pair of its strip in its own LDS, plainly
// read, added and written, without atomics: the coordinate moves by at least
// 1 / P of a bin per pixel, so no strip holds pixels P lanes apart.  For P = 2
// the first of two neighbours in one strip adds the other's terms to its own;
// beyond, the lanes of one residue mod P go together, in P passes.  (A run that
// breaks the rule, as a fan's may at the edge, falls back to LDS atomics;
// within one wave those too come in a fixed order.)  Every pixel is evaluated
// once, where the strips above test two or three candidates for each that they
// hold, and once for NB items of a batch.  The waves of a workgroup share a view
// and meet in LDS in a fixed order.  Units of zeros are passed over after their
// loads (512^2, 360 views of one pixel: 64 us, of 251 dense); strips do not look
// for them, it costs dense data 5 to 20% there.
//
// Runs along y read a column, 64 cache lines for a wave; RUN_COLS neighbouring
// ones are read by wide loads, so that each line is touched twice and not once
// a run.  8 x 256^2, 360 parallel views: 252 us with four loads of a pixel
// each, 211 with one of four, 200 with two for eight runs and 150 with two items
// together, then bound by about 31 vector operations for each pixel and item (0.9
// a clock and CU).
constexpr int RUN_COLS = 8;          // runs whose pixels are loaded together
constexpr size_t RUN_LDS = 65536;    // LDS of a workgroup, at most

template <typename TI, bool FAN, int P, int NB>
__global__ void __launch_bounds__(1024) bpT2d_run_kernel(Geom2D g, const float2 *__restrict__ views,
                                                         const TI *__restrict__ img, float *__restrict__ sino,
                                                         int batch, unsigned block0)
{
    typedef float Pairs __attribute__((ext_vector_type(2 * NB)));   // (w0, w1) of each item
    extern __shared__ __align__(32) char run_lds[];   // g.nu + 1 strips (-1 .. nu - 1) per wave
    Pairs *part = (Pairs *)run_lds;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int waves = blockDim.x >> 6, strips = g.nu + 1;
    const unsigned block = block0 + blockIdx.x;
    const int k = (int)(block % (unsigned)g.n_proj), b0 = NB * (int)(block / (unsigned)g.n_proj);
    const float2 c = views[k];
    const size_t pixels = (size_t)g.nx * g.ny;
    Pairs *own = part + wave * strips;
    for (int n = lane; n < strips; n += 64)
        own[n] = 0.0f;
    wave_lds_fence();
    // runs along x (rows of the image), or along y
    const bool along_x = fabsf(c.y) * g.sx >= fabsf(c.x) * g.sy;
    const int nq = along_x ? g.nx : g.ny, np = along_x ? g.ny : g.nx;
    const int chunks = (nq + 63) / 64, groups = (np + RUN_COLS - 1) / RUN_COLS;
    // units of RUN_COLS runs of one chunk; a wave's units are spread so that
    // the workgroup's waves read the same cache lines when runs go along y
    for (int u = wave; u < chunks * groups; u += waves) {
        const int q = u / groups * 64 + lane, p0 = u % groups * RUN_COLS;
        const int qc = min(q, nq - 1);
        float val[NB][RUN_COLS];
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const TI *im = img + (size_t)min(b0 + i, batch - 1) * pixels;
            if (!along_x && p0 + RUN_COLS <= np) {
                TI row[RUN_COLS];   // wide loads: the lanes lie on 64 cache lines
                __builtin_memcpy(row, im + ((size_t)qc * g.nx + p0), sizeof row);
#pragma unroll
                for (int r = 0; r < RUN_COLS; ++r)
                    val[i][r] = load_f32(&row[r]);
            } else {
#pragma unroll
                for (int r = 0; r < RUN_COLS; ++r) {
                    const int pc = min(p0 + r, np - 1);
                    val[i][r] = load_f32(im + (along_x ? (size_t)pc * g.nx + qc : (size_t)qc * g.nx + pc));
                }
            }
        }
        unsigned any = 0;
#pragma unroll
        for (int i = 0; i < NB; ++i)
#pragma unroll
            for (int r = 0; r < RUN_COLS; ++r)
                any |= __float_as_uint(val[i][r]);
        if (!__any(any))
            continue;   // zeros add nothing
        with_form<FAN>(g, [&](auto form) {
#pragma unroll
            for (int r = 0; r < RUN_COLS; ++r) {
                const int p = p0 + r;
                if (p >= np)   // uniform
                    break;
                const float x = fmaf((float)(along_x ? qc : p), g.sx, g.ox), y = fmaf((float)(along_x ? p : qc), g.sy, g.oy);
                float fu, t, wt;
                point2d<FAN, decltype(form)::value>(g, c, x, y, fu, t, wt);
                Pairs w;
#pragma unroll
                for (int i = 0; i < NB; ++i) {
                    const float v = FAN ? wt * val[i][r] : val[i][r];
                    w[2 * i] = v * (1.0f - t);
                    w[2 * i + 1] = v * t;
                }
                // strips -1 .. nu - 1; the rest of the lanes, and those past the run, add nothing
                const bool used = q < nq && fu >= -1.0f && fu < (float)g.nu;
                const int n = used ? (int)fu + 1 : -1;
                // the strips of the next lane and the one after it, or P lanes on
                const int next = next_lane(n, -2), far = P == 1 ? next : P == 2 ? next_lane(next, -2) : __shfl_down(n, P);
                if (__any(used && far == n && (P <= 2 || lane + P < 64))) {
                    if (used) {
#pragma unroll
                        for (int i = 0; i < 2 * NB; ++i)
                            unsafeAtomicAdd((float *)(own + n) + i, w[i]);
                    }
                    continue;
                }
                if constexpr (P <= 2) {
                    bool first = used;   // holds its strip's sum
                    if constexpr (P == 2) {
#pragma unroll
                        for (int i = 0; i < 2 * NB; ++i) {
                            const float o = next_lane(w[i], 0.0f);
                            w[i] += next == n ? o : 0.0f;
                        }
                        first = used && prev_lane(n, -2) != n;
                    }
                    if (first)
                        own[n] += w;
                } else {
#pragma unroll
                    for (int h = 0; h < P; ++h) {
                        if (used && lane % P == h)
                            own[n] += w;
                        __builtin_amdgcn_wave_barrier();
                    }
                }
                __builtin_amdgcn_wave_barrier();
            }
        });
    }
    __syncthreads();
    for (int j = threadIdx.x; j < g.nu; j += blockDim.x) {
        float s0[NB], s1[NB];
#pragma unroll
        for (int i = 0; i < NB; ++i)
            s0[i] = s1[i] = 0.0f;
        for (int w = 0; w < waves; ++w) {
            const Pairs above = part[w * strips + j + 1], below = part[w * strips + j];
#pragma unroll
            for (int i = 0; i < NB; ++i) {
                s0[i] += above[2 * i];
                s1[i] += below[2 * i + 1];
            }
        }
#pragma unroll
        for (int i = 0; i < NB; ++i)
            if (b0 + i < batch)
                sino[((size_t)(b0 + i) * g.n_proj + k) * g.nu + j] = g.dbeta * (s0[i] + s1[i]);
    }
}

template <typename T, typename TI, bool FAN, int V, int NB, int PX = 8>
hipError_t fpT2d_n(const Geom2D &g, const float2 *views, const void *sino, void *img, int batch, hipStream_t s)
{
    const int ntx = (g.nx + PX - 1) / PX, nty = (g.ny + PX - 1) / PX;
    const long tiles = (long)ntx * nty * ((batch + NB - 1) / NB);
    // waves per tile: about 32 on every CU in all, at least V views each (a
    // small image's time is one wave's chain of views: 256^2 with 30 views, 15.0
    // us for four waves of eight views, 13.2 us for eight of four)
    long waves = (8192 + tiles - 1) / tiles;
    const long most = (g.n_proj + V - 1) / V;
    waves = waves < most ? waves : most;
    waves = waves < 16 ? waves : 16;
    const int threads = (int)(64 * waves);
    return launch_in_pieces(tiles, threads, [&](unsigned first, dim3 grid) {
        hipLaunchKernelGGL((fpT2d_kernel<T, TI, FAN, V, NB, PX>), grid, dim3(threads), threads * sizeof(TileRay<NB>), s, g,
                           views, (const TI *)sino, (T *)img, ntx, nty, batch, first);
    });
}

template <typename T, typename TI, bool FAN, int V>
hipError_t fpT2d_v(const Geom2D &g, const float2 *views, const void *sino, void *img, int batch, hipStream_t s)
{
    // up to eight items of a batch share the rays and weights (512^2, 360 fan
    // views of 1020 bins, two and five items: 1526 and 3439 us one at a time, 828
    // and 2201 by twos, 1581 five by fours, 1046 in one; 64^2, 90 parallel views of
    // five: 18, 12, 13 and 14 us)
    if (batch > 4)
        return fpT2d_n<T, TI, FAN, V, 8>(g, views, sino, img, batch, s);
    if (batch > 2)
        return fpT2d_n<T, TI, FAN, V, 4>(g, views, sino, img, batch, s);
    return batch == 2 ? fpT2d_n<T, TI, FAN, V, 2>(g, views, sino, img, batch, s)
                      : fpT2d_n<T, TI, FAN, V, 1>(g, views, sino, img, batch, s);
}

template <typename T, typename TI, bool FAN>
hipError_t fpT2d_f(const Geom2D &g, const float2 *views, const void *sino, void *img, int batch, hipStream_t s)
{
    // Tiles of 4 x 4 pixels where those of 8 x 8 leave half of the CUs without
    // one: their waves are chains of views (one item, 200 parallel and fan views,
    // us for tiles of eight and four: 32^2 22.5 and 9.9, 33.2 and 13.5; 64^2 22.2 and
    // 10.9, 33.6 and 14.6; 80^2 22.3 and 15.1, 33.6 and 24.8; 96^2 22.3 and 20.4, 34.4
    // and 36.5; three items of 48^2 23.8 and 15.6, 36.2 and 25.9, of 64^2 23.7 and
    // 22.3, 35.8 and 41.1).
    if ((long)((g.nx + 7) / 8) * ((g.ny + 7) / 8) * batch <= 128)
        return fpT2d_n<T, TI, FAN, 4, 1, 4>(g, views, sino, img, batch, s);
    // Views set up together, so that the rays of an 8 x 8 tile's support at the
    // isocentre (its diagonal and three bins for the rounded-out ends) fill the
    // wave; a view that needs more lanes is set up in several passes.  512^2,
    // 360 fan views, 13 bins, with A: 1.17, 0.95 and 0.89 ms for one, two and four views.
    const float diag = 9.0f * sqrtf(g.sx * g.sx + g.sy * g.sy), n = diag * (FAN ? g.ru / g.sid : g.ru) + 3.0f;
    if (n <= 16.0f)
        return fpT2d_v<T, TI, FAN, 4>(g, views, sino, img, batch, s);
    if (n <= 32.0f)
        return fpT2d_v<T, TI, FAN, 2>(g, views, sino, img, batch, s);
    return fpT2d_v<T, TI, FAN, 1>(g, views, sino, img, batch, s);
}

template <typename T, typename TI>
hipError_t fpT2d(bool fan, const Geom2D &g, const float2 *views, const void *sino, void *img, int batch,
                 hipStream_t s)
{
    return fan ? fpT2d_f<T, TI, true>(g, views, sino, img, batch, s)
               : fpT2d_f<T, TI, false>(g, views, sino, img, batch, s);
}

template <typename T, int AT_T, int AT_RAYS>
hipError_t fpT_cone_t(const Geom3D &g, const ConeFPView *fviews, const ConeBPView *bviews, const void *proj, void *vol,
                      int batch, double *part, int shares, hipStream_t s)
{
    const int nbx = (g.nx + AT_B - 1) / AT_B, nby = (g.ny + AT_B - 1) / AT_B, nbz = (g.nz + AT_B - 1) / AT_B;
    const long blocks = (long)nbx * nby * nbz * batch;
    // (shares only where there are few bricks: one piece)
    const hipError_t e = launch_in_pieces(blocks, AT_T, [&](unsigned first, dim3 grid) {
        grid.y = (unsigned)shares;
        hipLaunchKernelGGL((fpT_cone_kernel<T, T, AT_T, AT_RAYS>), grid, dim3(AT_T), 0, s, g, fviews, bviews,
                           (const T *)proj, (T *)vol, shares > 1 ? part : nullptr, nbx, nby, nbz, first);
    });
    if (e != hipSuccess || shares == 1)
        return e;
    hipLaunchKernelGGL((fpT_cone_sum_kernel<T, AT_T>), dim3((unsigned)blocks * (AT_B * AT_B * AT_B / 256)), dim3(256), 0,
                       s, g, part, (T *)vol, nbx, nby, nbz, shares, (unsigned)blocks);
    return hipGetLastError();
}

template <typename T>
hipError_t fpT_cone(const Geom3D &g, const ConeFPView *fviews, const ConeBPView *bviews, const void *proj, void *vol,
                    int batch, double *part, int shares, hipStream_t s)
{
    // A footprint (at the isocentre, with the corners' roundings) of few rays keeps
    // few of 512 threads busy: 256^3, 40 views, ms with 512 and 256 threads for
    // footprints of 1121, 700, 487, 333 and 174 rays 8.33 and 7.98, 4.85 and 5.13, 3.63
    // and 3.29, 3.08 and 2.36, 2.76 and 1.84; 41^3, 60 views, us 196 and 216, 131 and
    // 144, 91 and 128, 76 and 73, 71 and 66.
    const float mag = g.sdd / g.sid;
    const float rays = ((float)AT_B * sqrtf(g.sx * g.sx + g.sy * g.sy) * mag / g.du + 3.0f) *
                       ((float)AT_B * g.sz * mag / g.dv + 3.0f);
    if (rays <= 400.0f)
        return fpT_cone_t<T, 256, 640>(g, fviews, bviews, proj, vol, batch, part, shares, s);
    return fpT_cone_t<T, 512, 1024>(g, fviews, bviews, proj, vol, batch, part, shares, s);
}

}  // namespace

template <typename T>
__global__ void cast_kernel(const float *__restrict__ in, T *__restrict__ out, size_t n)
{
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        store_f32(out + i, in[i]);
}

hipError_t launch_cast_from_f32(int dtype, const float *in, void *out, size_t n, hipStream_t s)
{
    const size_t blocks = (n + 255) / 256;
    const dim3 grid((unsigned)(blocks < 4096 ? blocks : 4096));
    switch (dtype) {
    case 1: hipLaunchKernelGGL(cast_kernel<f16_t>, grid, dim3(256), 0, s, in, (f16_t *)out, n); break;
    case 2: hipLaunchKernelGGL(cast_kernel<bf16_t>, grid, dim3(256), 0, s, in, (bf16_t *)out, n); break;
    default: hipLaunchKernelGGL(cast_kernel<float>, grid, dim3(256), 0, s, in, (float *)out, n); break;
    }
    return hipGetLastError();
}

hipError_t fill_zero(float *p, size_t n, hipStream_t s)
{
    const size_t blocks = (n + 255) / 256;
    hipLaunchKernelGGL(fill_zero_kernel, dim3((unsigned)(blocks < 4096 ? blocks : 4096)), dim3(256), 0, s, p, n);
    return hipGetLastError();
}

hipError_t launch_project_adjoint_2d(int dtype, bool fan, const Geom2D &g, const float2 *views, const void *sino,
                                     void *img, int batch, hipStream_t stream)
{
    switch (dtype) {
    case 0: return fpT2d<float, float>(fan, g, views, sino, img, batch, stream);
    case 1: return fpT2d<f16_t, f16_t>(fan, g, views, sino, img, batch, stream);
    default: return fpT2d<bf16_t, bf16_t>(fan, g, views, sino, img, batch, stream);
    }
}

static size_t at_bricks(const Geom3D &g, int batch)
{
    const size_t n = AT_B;
    return ((size_t)g.nx + n - 1) / n * (((size_t)g.ny + n - 1) / n) * (((size_t)g.nz + n - 1) / n) * (size_t)batch;
}

// Shares of the views: 512 workgroups are resident at a time, and four times
// as many even out their lengths (128^3, 124 views: 6.50, 6.28, 6.04 and
// 5.97 ms for 1, 2, 3 and 4 shares of 512 bricks, with A), but a share of a
// few views spends its time on partial sums (32^3, 360 views: 0.195, 0.209
// and 0.248 ms for 64, 128 and 256 shares of 8 bricks).
static int at_shares(const Geom3D &g, int batch)
{
    const size_t bricks = at_bricks(g, batch), most = bricks < 2048 ? 2048 / bricks : 1;
    const size_t shares = most < (size_t)g.n_proj / 6 ? most : (size_t)g.n_proj / 6;
    return shares > 1 ? (int)shares : 1;
}

size_t project_adjoint_scratch(const Geom3D &g, int batch)
{
    const int shares = at_shares(g, batch);
    return shares > 1 ? at_bricks(g, batch) * (size_t)shares * (AT_B * AT_B * AT_B * sizeof(double)) : 0;
}

hipError_t launch_project_adjoint_cone(int dtype, const Geom3D &g, const ConeFPView *fviews,
                                       const ConeBPView *bviews, const void *proj, void *vol, int batch,
                                       double *scratch, hipStream_t stream)
{
    const int shares = scratch ? at_shares(g, batch) : 1;
    switch (dtype) {
    case 0: return fpT_cone<float>(g, fviews, bviews, proj, vol, batch, scratch, shares, stream);
    case 1: return fpT_cone<f16_t>(g, fviews, bviews, proj, vol, batch, scratch, shares, stream);
    default: return fpT_cone<bf16_t>(g, fviews, bviews, proj, vol, batch, scratch, shares, stream);
    }
}

template <typename TI, int P, int NB>
hipError_t bpT2d_run(bool fan, const Geom2D &g, const float2 *views, const void *img, float *sino, int batch,
                     hipStream_t stream)
{
    const long groups = (long)g.n_proj * ((batch + NB - 1) / NB);
    const size_t bins = (size_t)(g.nu + 1) * NB * sizeof(float2);   // LDS per wave
    int waves = 1;
    while (waves < 16 && groups * waves < 16384 && 2 * waves * bins <= RUN_LDS)
        waves *= 2;
    const dim3 block(64 * waves);
    const size_t lds = (size_t)waves * bins;
    return launch_in_pieces(groups, 64 * waves, [&](unsigned first, dim3 grid) {
        if (fan)
            hipLaunchKernelGGL((bpT2d_run_kernel<TI, true, P, NB>), grid, block, lds, stream, g, views, (const TI *)img,
                               sino, batch, first);
        else
            hipLaunchKernelGGL((bpT2d_run_kernel<TI, false, P, NB>), grid, block, lds, stream, g, views,
                               (const TI *)img, sino, batch, first);
    });
}

template <typename TI, int P>
hipError_t bpT2d_run_p(int nb, bool fan, const Geom2D &g, const float2 *views, const void *img, float *sino, int batch,
                       hipStream_t stream)
{
    return nb == 2 ? bpT2d_run<TI, P, 2>(fan, g, views, img, sino, batch, stream)
                   : bpT2d_run<TI, P, 1>(fan, g, views, img, sino, batch, stream);
}

template <typename TI>
hipError_t bpT2d(bool fan, const Geom2D &g, const float2 *views, const void *img, float *sino, int batch,
                 hipStream_t stream)
{
    // Runs, where a view to a workgroup fills the GPU, and the pixels of a run
    // move by at least a quarter of a bin: the faster axis moves by 1 / sqrt(2) of a
    // spacing on the detector, seen from the far side of the image.  The larger a
    // view's work for its one workgroup (its pixels, in runs of whole waves), the
    // more views it takes: 0.55 sqrt(pixels), and any number up to 128^2, where the
    // sixteen waves have a few runs each.  Runs to strips break even at about (views
    // of one item, parallel, flat and arc): 128^2 none, 160^2 70, 45 and 45 (rule 97),
    // 256^2 60, 170 and 170 (141), 320^2 80, 185 and 140 (176), 512^2 230, 400 and 230
    // (282), 700^2 400, 450 and 256 (386).
    const float wx = g.nx * g.sx, wy = g.ny * g.sy;
    const float rate = 0.7071f * fminf(g.sx, g.sy) * (fan ? g.ru / (g.sid + 0.5f * sqrtf(wx * wx + wy * wy)) : g.ru);
    const int P = rate >= 1.0f ? 1 : rate >= 0.5f ? 2 : rate >= 0.3334f ? 3 : rate >= 0.25f ? 4 : 0;
    const long items = (long)g.n_proj * batch;
    const size_t bins = (size_t)(g.nu + 1) * sizeof(float2);   // LDS per wave and item
    // Two items of a batch together, where eight waves of a workgroup still find
    // LDS and the chip is filled (parallel, 256^2: 180 views of 2 and 5 items and
    // 360 of 8: 43, 76 and 200 us alone, 52, 75 and 155 by twos; 512^2, 360 fan
    // views of 1020 bins, four waves to a workgroup: 382 and 452).
    const int nb = batch > 1 && 16 * bins <= RUN_LDS && (long)g.n_proj * ((batch + 1) / 2) >= 512 ? 2 : 1;
    const float pixels = 32.0f * ((float)((g.nx + 63) / 64) * g.ny + (float)((g.ny + 63) / 64) * g.nx);
    if (P > 0 && bins <= RUN_LDS && (pixels <= 16384.0f || (float)items >= 0.55f * sqrtf(pixels))) {
        switch (P) {
        case 1: return bpT2d_run_p<TI, 1>(nb, fan, g, views, img, sino, batch, stream);
        case 2: return bpT2d_run_p<TI, 2>(nb, fan, g, views, img, sino, batch, stream);
        case 3: return bpT2d_run_p<TI, 3>(nb, fan, g, views, img, sino, batch, stream);
        default: return bpT2d_run_p<TI, 4>(nb, fan, g, views, img, sino, batch, stream);
        }
    }
    const int groups = (g.nu + 62) / 63;
    const long blocks = (long)groups * g.n_proj * batch;
    // waves per workgroup: enough for about 16 waves on every CU, at least
    // eight rows each
    int waves = 1;
    while (waves < 16 && blocks * waves < 4096 && waves * 16 <= (g.nx < g.ny ? g.nx : g.ny))
        waves *= 2;
    const dim3 block(64 * waves);
    const size_t lds = waves > 1 ? 64 * waves * sizeof(float2) : 0;
    return launch_in_pieces(blocks, 64 * waves, [&](unsigned first, dim3 grid) {
        if (fan)
            hipLaunchKernelGGL((bpT2d_kernel<TI, true>), grid, block, lds, stream, g, views, (const TI *)img, sino,
                               groups, first);
        else
            hipLaunchKernelGGL((bpT2d_kernel<TI, false>), grid, block, lds, stream, g, views, (const TI *)img, sino,
                               groups, first);
    });
}

hipError_t launch_backproject_adjoint_2d(int in_dtype, bool fan, const Geom2D &g, const float2 *views,
                                         const void *img, float *sino, int batch, hipStream_t stream)
{
    switch (in_dtype) {
    case 0: return bpT2d<float>(fan, g, views, img, sino, batch, stream);
    case 1: return bpT2d<f16_t>(fan, g, views, img, sino, batch, stream);
    default: return bpT2d<bf16_t>(fan, g, views, img, sino, batch, stream);
    }
}

}  // namespace ph
