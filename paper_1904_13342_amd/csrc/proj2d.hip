// 2D parallel- and fan-beam forward projection (ray-driven, a few lanes per
// detector bin) and back-projection (voxel-driven, a few waves per 8 x 8 pixels),
// Sec. II.B.2.  The images of the 2D workloads (at most 512 x 512 FP32,
// 1 MiB) stay resident in L2; what neighbouring rays or pixels share, A in slabs
// and B in segments stage once more in LDS.
#include "device_util.h"
#include "ranges.h"

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

// Bilinear sample at (X, Y), zero outside the image.
template <typename T>
__device__ __forceinline__ float sample_direct(const T *im, const Geom2D &g, float X, float Y)
{
    const float fx = floorf(X), fy = floorf(Y);
    const int ix = (int)fx, iy = (int)fy;
    const float tx = X - fx, ty = Y - fy;
    const float p00 = pix(im, g.nx, g.ny, ix, iy), p01 = pix(im, g.nx, g.ny, ix + 1, iy);
    const float p10 = pix(im, g.nx, g.ny, ix, iy + 1), p11 = pix(im, g.nx, g.ny, ix + 1, iy + 1);
    const float a0 = fmaf(tx, p01 - p00, p00), a1 = fmaf(tx, p11 - p10, p10);
    return fmaf(ty, a1 - a0, a0);
}

constexpr int A_UNROLL = 2;   // samples per lane of A whose loads are in flight together
constexpr int B_UNROLL = 4;   // views per wave of B

// S lanes share one ray (S a power of two, at most 64: the lanes of a ray lie
// in one wave); lane s takes samples k0 + s, k0 + s + S, ... and the partial
// sums meet in a fixed shuffle tree.  Small problems (few rays, long rays)
// then still fill the machine.
//
// A lane takes two samples at a time (four or eight leave more of a short ray
// to its checked ends).  Where every sample of the wave's two
// has its 2 x 2 cell inside the image (all but a ray's ends), the cell is
// read as two pairs at 32-bit offsets from the image, without bounds checks:
// 17 vector operations and two loads a sample.  Elsewhere the four pixels
// are read at clamped indices and masked.  (Four conditional loads per
// sample, each in a branch of its own, took 0.60 ms for 512^2 and 360 fan
// views of 725 bins; this takes 0.32 ms, bound by the scattered loads, about
// 40 clocks per CU for each.)  Taken for few rays, for bins much wider than
// a pixel and for steps longer than one; the rest goes in slabs, below.
template <typename T, bool FAN, int S>
__global__ void __launch_bounds__(256) fp2d_kernel(Geom2D g, const float2 *__restrict__ views,
                                                   const T *__restrict__ img, T *__restrict__ sino, unsigned n_rays,
                                                   unsigned blocks, unsigned block0)
{
    const unsigned block = block0 + blockIdx.x;
    const int b = (int)(block / blocks);
    const long t = (long)(block % blocks) * 256 + threadIdx.x;
    const unsigned r = (unsigned)(t / S);
    const int s = (int)(t % S);
    if (r >= n_rays)
        return;   // whole rays only: the S lanes of a ray leave together
    const int j = (int)(r % (unsigned)g.nu), k = (int)(r / (unsigned)g.nu);
    const T *im = img + (size_t)b * g.nx * g.ny, *im1 = im + g.nx;
    float X0, Y0, eX, eY;
    make_ray_2d<FAN>(g, views[k], j, X0, Y0, eX, eY);
    float lo = -3.0e38f, hi = 3.0e38f;
    float acc = 0.0f;
    if (krange(X0, eX, -1.0f, (float)g.nx, lo, hi) && krange(Y0, eY, -1.0f, (float)g.ny, lo, hi) && lo < hi) {
        const int k0 = (int)floorf(lo) - 1, k1 = (int)ceilf(hi) + 1;
        int in_lo, in_hi;   // samples whose cells lie inside the image
        cell_range(X0, Y0, eX, eY, g.nx, g.ny, sizeof(T), in_lo, in_hi);
        for (int m = k0 + s; m <= k1; m += A_UNROLL * S) {
            if (__all(m >= in_lo && m + (A_UNROLL - 1) * S <= in_hi)) {
                float2 p[A_UNROLL], q[A_UNROLL];
                float tx[A_UNROLL], ty[A_UNROLL];
#pragma unroll
                for (int u = 0; u < A_UNROLL; ++u) {
                    const float fm = (float)(m + u * S), X = fmaf(fm, eX, X0), Y = fmaf(fm, eY, Y0);
                    tx[u] = __builtin_amdgcn_fractf(X);
                    ty[u] = __builtin_amdgcn_fractf(Y);
                    const unsigned off = (__umul24((unsigned)Y, (unsigned)g.nx) + (unsigned)X) * (unsigned)sizeof(T);
                    p[u] = load_pair(im, off);
                    q[u] = load_pair(im1, off);
                }
#pragma unroll
                for (int u = 0; u < A_UNROLL; ++u) {
                    const float a0 = fmaf(tx[u], p[u].y - p[u].x, p[u].x), a1 = fmaf(tx[u], q[u].y - q[u].x, q[u].x);
                    acc += fmaf(ty[u], a1 - a0, a0);
                }
            } else {
#pragma unroll
                for (int u = 0; u < A_UNROLL; ++u) {
                    const float fm = (float)(m + u * S);
                    const float v = sample_direct(im, g, fmaf(fm, eX, X0), fmaf(fm, eY, Y0));
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

// The same operator in slabs.  A wave holds 64 neighbouring rays of one view,
// which advance together along axis A (x or y, the one its slowest ray advances
// faster on).  The image is walked in slabs of SL_D planes across A; each slab's
// cross-section, between the wave's two outer rays and a pixel of margin, is
// loaded into registers while the slab before it is sampled, then written to
// the wave's own LDS, and every ray takes the samples whose floor(A) falls in
// the slab, two ds_read2 each.  Loads are one contiguous run per row (A = y) or
// eight rows of eight pixels (A = x), where the direct kernel's touch a cache
// line for every few lanes.  The W waves of a workgroup share the rays, each
// taking a run of slabs, and meet in LDS in a fixed order.
// Positions and interpolation are those of the direct kernel bit for bit.
// 512^2, 360 fan views of 725 bins: 0.32 -> 0.17 ms (0.9 Tsamples/s).  34 lane
// operations a sample, 0.76 instructions a clock and CU; bank conflicts of the
// reads keep the LDS for another quarter of the time.
constexpr int SL_D = 7;          // planes a slab advances
constexpr int SL_P = SL_D + 1;   // planes it holds
constexpr size_t SL_LDS = 65536;   // LDS of a workgroup, at most

__device__ __forceinline__ int floor_int(float x)
{
    int r;
    asm("v_cvt_flr_i32_f32 %0, %1" : "=v"(r) : "v"(x));
    return r;
}

__device__ __forceinline__ float lane_value(float x, int lane)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x), lane));
}

// One wave's share of the slabs; SW the row pitch in words (and the widest
// slab), 8 mod 32 so that the writes of eight rows by eight pixels spread over
// the banks.
template <typename T, int AX, int SW>
__device__ __forceinline__ float slab_walk_2d(const Geom2D &g, const T *im, float *slab, float X0, float Y0, float eX,
                                              float eY, bool hit, int kb, int ke, int last, int lane, int wave,
                                              int waves)
{
    constexpr int NB_LOADS = AX == 1 ? (SW + 63) / 64 * SL_P : (SW + 7) / 8;
    const int NB = AX == 0 ? g.ny : g.nx;
    const float PA = AX == 0 ? X0 : Y0, eA = AX == 0 ? eX : eY, PB = AX == 0 ? Y0 : X0, eB = AX == 0 ? eY : eX;
    const bool up = lane_value(eA, 0) > 0.0f;
    const float rEA = 1.0f / eA, slope = eB * rEA;
    // the outer rays, B = b0 + A slope
    const float s0 = lane_value(slope, 0), s1 = lane_value(slope, last);
    const float b0 = lane_value(fmaf(-PA, slope, PB), 0), b1 = lane_value(fmaf(-PA, slope, PB), last);
    // slab s holds floor(A) in [-2 + s D, -2 + (s + 1) D)
    int s_min = 1 << 30, s_max = -1;
    if (hit) {
        const int ia = floor_int(fmaf((float)kb, eA, PA)), ie = floor_int(fmaf((float)ke, eA, PA));
        s_min = (min(ia, ie) + 2) / SL_D;
        s_max = (max(ia, ie) + 2) / SL_D;
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        s_min = min(s_min, __shfl_xor(s_min, o));
        s_max = max(s_max, __shfl_xor(s_max, o));
    }
    s_min = __builtin_amdgcn_readfirstlane(s_min);
    s_max = __builtin_amdgcn_readfirstlane(s_max);
    if (s_max < s_min)
        return 0.0f;   // no ray of the wave meets the image
    const int n_all = s_max - s_min + 1;
    const int n0 = n_all * wave / waves, n1 = n_all * (wave + 1) / waves;   // this wave's slabs
    if (n1 <= n0)
        return 0.0f;
    auto first_plane = [&](int n) { return -2 + SL_D * (up ? s_min + n : s_max - n); };
    struct Box {
        int a0, b_lo, w;
    };
    auto box_of = [&](int n) {
        Box x;
        x.a0 = first_plane(n);
        const float a = (float)x.a0, e = (float)(x.a0 + SL_D);
        const float p0 = fmaf(a, s0, b0), p1 = fmaf(e, s0, b0), p2 = fmaf(a, s1, b1), p3 = fmaf(e, s1, b1);
        const float lo = fminf(fminf(p0, p1), fminf(p2, p3)), hi = fmaxf(fmaxf(p0, p1), fmaxf(p2, p3));
        const int l = max(floor_int(lo) - 1, -2), h = min(floor_int(hi) + 2, NB + 1);
        x.b_lo = __builtin_amdgcn_readfirstlane(l);
        x.w = __builtin_amdgcn_readfirstlane(h) - x.b_lo + 1;
        return x;
    };
    float buf[NB_LOADS];
    auto load = [&](const Box &x) {
        if (x.w > SW || x.w <= 0)
            return;
        if (AX == 1) {   // rows of the image
#pragma unroll
            for (int c = 0; c < (SW + 63) / 64; ++c) {
                const int gx = x.b_lo + 64 * c + lane, cx = min(max(gx, 0), g.nx - 1);
                const bool okx = cx == gx && 64 * c + lane < x.w;
                if (64 * c < x.w) {   // uniform
#pragma unroll
                    for (int p = 0; p < SL_P; ++p) {
                        const int gy = x.a0 + p, cy = min(max(gy, 0), g.ny - 1);   // uniform
                        const float v = load_f32(im + (size_t)cy * g.nx + cx);
                        buf[c * SL_P + p] = okx && cy == gy ? v : 0.0f;
                    }
                }
            }
        } else {   // eight pixels of eight rows at a time
            const int gx = x.a0 + (lane & 7), cx = min(max(gx, 0), g.nx - 1);
#pragma unroll
            for (int i = 0; i < NB_LOADS; ++i) {
                if (8 * i < x.w) {   // uniform
                    const int gy = x.b_lo + 8 * i + (lane >> 3), cy = min(max(gy, 0), g.ny - 1);
                    const float v = load_f32(im + (size_t)cy * g.nx + cx);
                    buf[i] = cx == gx && cy == gy ? v : 0.0f;
                }
            }
        }
    };
    auto store = [&](const Box &x) {
        if (x.w > SW || x.w <= 0)
            return;
        if (AX == 1) {
#pragma unroll
            for (int c = 0; c < (SW + 63) / 64; ++c) {
                if (64 * c < x.w && 64 * c + lane < SW) {
#pragma unroll
                    for (int p = 0; p < SL_P; ++p)
                        slab[p * SW + 64 * c + lane] = buf[c * SL_P + p];
                }
            }
        } else {
#pragma unroll
            for (int i = 0; i < NB_LOADS; ++i)
                if (8 * i < x.w)
                    slab[(lane & 7) * SW + 8 * i + (lane >> 3)] = buf[i];
        }
    };

    Box cur = box_of(n0);
    load(cur);
    // this ray's first sample in the wave's slabs, counted with the coordinate
    // the slabs are told by: near its first sample of all (a margin sample may
    // round to just outside the first slab), or near the plane that the wave's
    // share begins at
    int m = kb;
    if (hit) {
        const float plane = (float)(up ? cur.a0 : cur.a0 + SL_D);
        if (n0 > 0)
            m = min(max((int)ceilf((plane - PA) * rEA), kb), ke + 1);
        auto before = [&](int q) {   // sample q lies in an earlier slab
            const int a = floor_int(fmaf((float)q, eA, PA));
            return up ? a < cur.a0 : a >= cur.a0 + SL_D;
        };
#pragma clang loop unroll(disable) vectorize(disable) interleave(disable)
        while (m <= ke && before(m))
            ++m;
#pragma clang loop unroll(disable) vectorize(disable) interleave(disable)
        while (m > kb && !before(m - 1))
            --m;
    }
    float acc = 0.0f;
    for (int n = n0; n < n1; ++n) {
        wave_lds_fence();   // the slab before this one has been sampled
        store(cur);
        wave_lds_fence();
        const Box x = cur;
        if (n + 1 < n1) {
            cur = box_of(n + 1);
            load(cur);
        }
        if (!hit)
            continue;
        auto in_slab = [&](int q) { return (unsigned)(floor_int(fmaf((float)q, eA, PA)) - x.a0) < (unsigned)SL_D; };
        int m_end = m;
        if (m <= ke && in_slab(m)) {
            const float bound = (float)(up ? x.a0 + SL_D : x.a0);
            m_end = sample_beyond(m, ke, bound, fmaf((float)m, eA, PA), rEA);
#pragma clang loop unroll(disable) vectorize(disable) interleave(disable)
            while (m_end > m + 1 && !in_slab(m_end - 1))
                --m_end;
#pragma clang loop unroll(disable) vectorize(disable) interleave(disable)
            while (m_end <= ke && in_slab(m_end))
                ++m_end;
        }
        if (x.w > 0 && x.w <= SW) {
            const int base = -4 * (x.a0 * SW + x.b_lo);
            auto sample = [&](float fm) {
                const float X = fmaf(fm, eX, X0), Y = fmaf(fm, eY, Y0);
                const float tx = __builtin_amdgcn_fractf(X), ty = __builtin_amdgcn_fractf(Y);
                const int iA = floor_int(AX == 0 ? X : Y), iB = floor_int(AX == 0 ? Y : X);
                const float *p = (const float *)((const char *)slab + (__mul24(iA, 4 * SW) + 4 * iB + base));
                const float p00 = p[0], p01 = AX == 1 ? p[1] : p[SW], p10 = AX == 1 ? p[SW] : p[1], p11 = p[SW + 1];
                const float a0 = fmaf(tx, p01 - p00, p00), a1 = fmaf(tx, p11 - p10, p10);
                return fmaf(ty, a1 - a0, a0);
            };
            // the slab's samples are summed first, so that no long sum is rounded at every sample
            const float fend = (float)m_end;
            float fm = (float)m, sum = 0.0f;
            for (; fm + 1.0f < fend; fm += 2.0f)
                sum += sample(fm) + sample(fm + 1.0f);
            if (fm < fend)
                sum += sample(fm);
            acc += sum;
        } else {
            for (int q = m; q < m_end; ++q)
                acc += sample_direct(im, g, fmaf((float)q, eX, X0), fmaf((float)q, eY, Y0));
        }
        m = m_end;
    }
    return acc;
}

template <typename T, bool FAN, int SW>
__global__ void __launch_bounds__(1024) fp2d_slab_kernel(Geom2D g, const float2 *__restrict__ views,
                                                         const T *__restrict__ img, T *__restrict__ sino, int groups,
                                                         unsigned block0)
{
    extern __shared__ float slabs[];   // SL_P * SW words per wave
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int waves = blockDim.x >> 6;
    const unsigned block = block0 + blockIdx.x;
    const int grp = (int)(block % (unsigned)groups);
    const long kb_ = block / (unsigned)groups;
    const int k = (int)(kb_ % g.n_proj), b = (int)(kb_ / g.n_proj);
    const int j = grp * 64 + lane, last = min(63, g.nu - 1 - grp * 64);
    const T *im = img + (size_t)b * g.nx * g.ny;
    float X0, Y0, eX, eY;
    make_ray_2d<FAN>(g, views[k], min(j, g.nu - 1), X0, Y0, eX, eY);
    float lo = -3.0e38f, hi = 3.0e38f;
    const bool hit = j < g.nu && krange(X0, eX, -1.0f, (float)g.nx, lo, hi) &&
                     krange(Y0, eY, -1.0f, (float)g.ny, lo, hi) && lo < hi;
    // one sample of margin on each side; samples outside the image add zeros
    const int kb = hit ? (int)floorf(lo) : 0, ke = hit ? (int)ceilf(hi) : -1;
    float mx = fabsf(eX), my = fabsf(eY);
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) {
        mx = fminf(mx, __shfl_xor(mx, o));
        my = fminf(my, __shfl_xor(my, o));
    }
    const int ax = __builtin_amdgcn_readfirstlane(mx >= my ? 0 : 1);
    // the walk needs all rays to advance one way along A, by at most a pixel a
    // step on both axes, and sample indices that are exact in FP32
    const float eA = ax == 0 ? eX : eY;
    const bool ok = __all(eA * lane_value(eA, 0) > 0.0f && fabsf(eX) <= 1.0f && fabsf(eY) <= 1.0f &&
                          abs(kb) < (1 << 23) && abs(ke) < (1 << 23));
    float acc = 0.0f;
    if (!ok) {
        for (int m = kb + wave; m <= ke; m += waves)
            acc += sample_direct(im, g, fmaf((float)m, eX, X0), fmaf((float)m, eY, Y0));
    } else if (ax == 0) {
        acc = slab_walk_2d<T, 0, SW>(g, im, slabs + wave * SL_P * SW, X0, Y0, eX, eY, hit, kb, ke, last, lane, wave,
                                     waves);
    } else {
        acc = slab_walk_2d<T, 1, SW>(g, im, slabs + wave * SL_P * SW, X0, Y0, eX, eY, hit, kb, ke, last, lane, wave,
                                     waves);
    }
    if (waves > 1) {
        __syncthreads();
        slabs[threadIdx.x] = acc;
        __syncthreads();
        if (wave > 0)
            return;
        for (int w = 1; w < waves; ++w)
            acc += slabs[w * 64 + lane];
    }
    if (j < g.nu)
        store_f32(sino + ((size_t)b * g.n_proj + k) * g.nu + j, g.step * acc);
}

// A wave owns a tile of 8 x 8 pixels and takes one view at a time, so the view
// is uniform and its 64 reads fall on a dozen neighbouring bins of one row.
// The W waves of a workgroup share a tile, wave w taking views w, w + W, ...,
// and meet in LDS in a fixed order.  Four views' loads are in flight together;
// where both bins of all four lie on the detector for the whole wave, each
// pair is one load, otherwise two masked ones.  (With the lanes of a wave on 4
// views of 16 pixels: 174 against 112 us for 8 x 256^2 and 360 parallel views.)
// Taken for single items of fan views, bound by the vector operations for each
// sample's coordinate, an atan2f on long arcs (512^2, 360 arc views of 725 bins: 53
// operations a sample in all, 1.1 a clock on every CU, 112 us), and for bins too
// fine to stage, below.
template <typename T, typename TI, bool FAN>
__global__ void __launch_bounds__(1024) bp2d_kernel(Geom2D g, const float2 *__restrict__ views,
                                                    const TI *__restrict__ sino, T *__restrict__ img, int ntx, int nty,
                                                    unsigned tile0)
{
    extern __shared__ float part[];   // one entry per thread, for more than one wave
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int waves = blockDim.x >> 6;
    const unsigned tile = tile0 + blockIdx.x;
    const int tx = (int)(tile % (unsigned)ntx), ty = (int)((tile / (unsigned)ntx) % (unsigned)nty);
    const int b = (int)(tile / ((unsigned)ntx * (unsigned)nty));
    const int ix = tx * 8 + (lane & 7), iy = ty * 8 + (lane >> 3);
    const TI *sb = sino + (size_t)b * g.n_proj * g.nu;
    const float x = fmaf((float)min(ix, g.nx - 1), g.sx, g.ox), y = fmaf((float)min(iy, g.ny - 1), g.sy, g.oy);
    float acc = 0.0f;
    for (int k0 = wave; k0 < g.n_proj; k0 += B_UNROLL * waves) {
        float fu[B_UNROLL], t[B_UNROLL], wt[B_UNROLL];
        bool inside = true;
        auto points = [&](auto form) {
#pragma unroll
            for (int u = 0; u < B_UNROLL; ++u) {
                const int k = min(k0 + u * waves, g.n_proj - 1);
                point2d<FAN, decltype(form)::value>(g, views[k], x, y, fu[u], t[u], wt[u]);
                inside = inside && fu[u] >= 0.0f && fu[u] < (float)(g.nu - 1);
            }
        };
        with_form<FAN>(g, points);
        if (__all(inside) && k0 + (B_UNROLL - 1) * waves < g.n_proj) {
            float2 p[B_UNROLL];
#pragma unroll
            for (int u = 0; u < B_UNROLL; ++u)
                p[u] = load_pair(sb + (size_t)(k0 + u * waves) * g.nu, (unsigned)fu[u] * (unsigned)sizeof(TI));
#pragma unroll
            for (int u = 0; u < B_UNROLL; ++u)
                acc = fmaf(wt[u], fmaf(t[u], p[u].y - p[u].x, p[u].x), acc);
        } else {
#pragma unroll
            for (int u = 0; u < B_UNROLL; ++u) {
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

// B in tiles of 16 x 16 pixels, four to a lane, for NB items of a batch at once.
// A wave takes a few views at a time: its lanes project the tile's four
// corners in each of them (the projection of a convex tile in front of the
// source is extreme at a corner) and stage the W bins from one below the
// lowest, zero outside the detector, in the wave's own LDS, the items of a bin
// side by side.  A pixel's coordinate is then found once for all items, and a
// sample is one read of a pair, with no bounds checks.  The next views' bins are
// loaded meanwhile.  A view whose corners span more bins than are staged, or lie
// so far out that FP32 bins round, is read from memory.  The waves of a
// workgroup share a tile and meet in LDS in a fixed order.  Reading pairs from
// memory cost about 25 clocks of a CU for each wave's sample; staged, it is 15
// vector operations, of which an item's own are three (8 x 256^2, 360 parallel
// views, with the launch: 122 us from memory, 88 staged one item at a time, 61 and
// 45 two and four, of which the kernel is 40).
constexpr int SB_BINS = 512;   // views times bins of a chunk

template <typename T, typename TI, bool FAN, int NB, int W>
__global__ void __launch_bounds__(1024) bp2d_seg_kernel(Geom2D g, const float2 *__restrict__ views,
                                                        const TI *__restrict__ sino, T *__restrict__ img, int ntx,
                                                        int nty, int batch, unsigned tile0)
{
    typedef float Items __attribute__((ext_vector_type(NB)));
    constexpr int LOADS = SB_BINS / 64, V = SB_BINS / W;   // V views to a chunk, at most one lane to a corner
    // SB_BINS of each wave, at the end its pixels' sums
    extern __shared__ __align__(16) char seg_lds[];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int waves = blockDim.x >> 6;
    const unsigned tile = tile0 + blockIdx.x;
    const int x0 = 16 * (int)(tile % (unsigned)ntx), y0 = 16 * (int)((tile / (unsigned)ntx) % (unsigned)nty);
    const int b0 = NB * (int)(tile / ((unsigned)ntx * (unsigned)nty));
    const size_t item = (size_t)g.n_proj * g.nu;
    Items *seg = (Items *)seg_lds + wave * SB_BINS;
    float px[2], py[2];
#pragma unroll
    for (int a = 0; a < 2; ++a) {
        px[a] = fmaf((float)min(x0 + 8 * a + (lane & 7), g.nx - 1), g.sx, g.ox);
        py[a] = fmaf((float)min(y0 + 8 * a + (lane >> 3), g.ny - 1), g.sy, g.oy);
    }
    // lane 4 v + c holds view v's corner c
    const float qx = fmaf((float)((lane & 1) ? min(x0 + 15, g.nx - 1) : x0), g.sx, g.ox);
    const float qy = fmaf((float)((lane & 2) ? min(y0 + 15, g.ny - 1) : y0), g.sy, g.oy);
    float2 cl, cl_next;   // view lane / 4, and its first staged bin
    int lo, lo_next;
    unsigned long long ok, ok_next, small, small_next;   // bit 4 v: view v is staged; its fan angles are small
    Items val[LOADS];
    auto fetch = [&](int k0) {
        const float2 c = cl_next = views[min(k0 + (lane >> 2), g.n_proj - 1)];
        float fu, t, wt;
        point2d<FAN, FORM_RANGE>(g, c, qx, qy, fu, t, wt);
        const float w = FAN ? fmaf(qx, c.x, fmaf(qy, c.y, g.sid)) : 1.0f;
        bool in = fabsf(fu) < 262144.0f;
        float mn = fu, mx = fu;
#pragma unroll
        for (int o = 1; o < 4; o <<= 1) {
            mn = fminf(mn, __shfl_xor(mn, o));
            mx = fmaxf(mx, __shfl_xor(mx, o));
        }
        in = in && mx - mn <= (float)(W - 4);   // one bin to each side, and the pair's second
        ok_next = __ballot(in);
        ok_next &= ok_next >> 1;
        ok_next &= ok_next >> 2;
        // below point2d's own bound by more than a rounding
        small_next = __ballot(fabsf(fmaf(qy, c.x, -(qx * c.y))) < 0.414f * w);
        small_next &= small_next >> 1;
        small_next &= small_next >> 2;
        lo_next = in ? (int)mn - 1 : 0;
#pragma unroll
        for (int i = 0; i < LOADS; ++i) {
            const int v = (64 * i + lane) / W;
            const int j = __shfl(lo_next, 4 * v) + lane % W, jc = min(max(j, 0), g.nu - 1);
            const TI *p = sino + (size_t)min(k0 + v, g.n_proj - 1) * g.nu + jc;
#pragma unroll
            for (int n = 0; n < NB; ++n) {
                const float q = load_f32(p + (size_t)min(b0 + n, batch - 1) * item);
                val[i][n] = j == jc ? q : 0.0f;
            }
        }
    };
    Items acc[4];
#pragma unroll
    for (int a = 0; a < 4; ++a)
        acc[a] = 0.0f;
    int k0 = wave * V;
    if (k0 < g.n_proj)
        fetch(k0);
    for (; k0 < g.n_proj; k0 += V * waves) {
        wave_lds_fence();   // the previous views have been read
#pragma unroll
        for (int i = 0; i < LOADS; ++i)
            seg[64 * i + lane] = val[i];
        wave_lds_fence();
        cl = cl_next;
        lo = lo_next;
        ok = ok_next;
        small = small_next;
        if (k0 + V * waves < g.n_proj)
            fetch(k0 + V * waves);
        const int nv = min(V, g.n_proj - k0);
        for (int v = 0; v < nv; ++v) {
            const float2 c = make_float2(lane_value(cl.x, 4 * v), lane_value(cl.y, 4 * v));
            float fu[4], t[4], wt[4];
            auto points = [&](auto form) {
#pragma unroll
                for (int a = 0; a < 4; ++a)
                    point2d<FAN, decltype(form)::value>(g, c, px[a & 1], py[a >> 1], fu[a], t[a], wt[a]);
            };
            if (FAN && g.curved && g.ru_lo != 0.0f && ((small >> (4 * v)) & 1))
                points(Form<FORM_FINE_ARC | FORM_SMALL>());
            else
                with_form<FAN>(g, points);
            if ((ok >> (4 * v)) & 1) {
                const int first = v * W - __builtin_amdgcn_readlane(lo, 4 * v);
#pragma unroll
                for (int a = 0; a < 4; ++a) {
                    const Items *p = seg + ((int)fu[a] + first);
                    const Items p0 = p[0], p1 = p[1];
#pragma unroll
                    for (int n = 0; n < NB; ++n)
                        acc[a][n] = fmaf(wt[a], fmaf(t[a], p1[n] - p0[n], p0[n]), acc[a][n]);
                }
            } else {
                const TI *row = sino + (size_t)(k0 + v) * g.nu;
#pragma unroll
                for (int a = 0; a < 4; ++a) {
                    const int j = (int)fu[a];
                    const int j0 = min(max(j, 0), g.nu - 1), j1 = min(max(j + 1, 0), g.nu - 1);
#pragma unroll
                    for (int n = 0; n < NB; ++n) {
                        const TI *q = row + (size_t)min(b0 + n, batch - 1) * item;
                        float p0 = load_f32(q + j0), p1 = load_f32(q + j1);
                        p0 = j0 == j ? p0 : 0.0f;
                        p1 = j1 == j + 1 ? p1 : 0.0f;
                        acc[a][n] = fmaf(wt[a], fmaf(t[a], p1 - p0, p0), acc[a][n]);
                    }
                }
            }
        }
    }
    if (waves > 1) {
        wave_lds_fence();
#pragma unroll
        for (int a = 0; a < 4; ++a)
            seg[64 * a + lane] = acc[a];
        __syncthreads();
        if (wave > 0)
            return;
        for (int w = 1; w < waves; ++w)
#pragma unroll
            for (int a = 0; a < 4; ++a)
                acc[a] += seg[w * SB_BINS + 64 * a + lane];
    }
#pragma unroll
    for (int a = 0; a < 4; ++a) {
        const int ix = x0 + 8 * (a & 1) + (lane & 7), iy = y0 + 8 * (a >> 1) + (lane >> 3);
        if (ix < g.nx && iy < g.ny)
#pragma unroll
            for (int n = 0; n < NB; ++n)
                if (b0 + n < batch)
                    store_f32(img + ((size_t)(b0 + n) * g.ny + iy) * g.nx + ix, g.dbeta * acc[a][n]);
    }
}

// Lanes per ray: up to about 2^21 threads in all, but at least 16 samples of
// the image's diagonal each, or setting the rays up outweighs sampling them
// (256^2, 30 parallel views: 16.2, 13.4, 13.6 and 16.0 us for at least 8, 16,
// 32 and 64 samples per lane; 64^2, 16 views 7.1, 7.1, 10.7 and 19.3 us).
inline int lanes_per_ray(const Geom2D &g, long rays)
{
    const float wx = g.nx * g.sx, wy = g.ny * g.sy, samples = sqrtf(wx * wx + wy * wy) / g.step;
    int S = 1;
    while (S < 64 && rays * S * 2 <= (1L << 21) && 32.0f * (float)S <= samples)
        S *= 2;
    return S;
}

template <typename T, bool FAN, int S>
hipError_t fp2d_s(const Geom2D &g, const float2 *views, const void *img, void *sino, int batch, hipStream_t s)
{
    const long n_rays = (long)g.nu * g.n_proj, blocks = (n_rays * S + 255) / 256;   // of one item
    if (n_rays > 0xffffffffL)
        return hipErrorInvalidConfiguration;
    return launch_in_pieces(blocks * batch, 256, [&](unsigned first, dim3 grid) {
        hipLaunchKernelGGL((fp2d_kernel<T, FAN, S>), grid, dim3(256), 0, s, g, views, (const T *)img, (T *)sino,
                           (unsigned)n_rays, (unsigned)blocks, first);
    });
}

template <typename T, bool FAN, int SW>
hipError_t fp2d_slab(const Geom2D &g, const float2 *views, const void *img, void *sino, int batch, hipStream_t s)
{
    const int groups = (g.nu + 63) / 64;
    const long blocks = (long)groups * g.n_proj * batch;
    // waves per 64 rays: about 64 on every CU in all (512^2, 360 fan views: 283,
    // 192, 161 and 160 us for 4096, 8192, 16384 and 32768 waves), at least
    // three slabs each along the mean of the image's sides (125 x 37, 500 fan
    // views: 37, 26 and 22 us by the shorter, the mean and the longer side; 430 x
    // 129, 48 views 32 and 54 by the shorter and the longer), and two workgroups
    // or more to a CU's LDS (the widest slabs, 512^2 and 60, 120 and 170 fan
    // views: 52, 88 and 120 us for the 16 waves of one workgroup, 45, 72 and 90
    // for at most eight)
    constexpr size_t slab = (size_t)SL_P * SW * sizeof(float);   // LDS of a wave
    int waves = 1;
    while (waves < 16 && blocks * waves < 16384 && 4 * waves * 3 * SL_D <= g.nx + g.ny &&
           2 * waves * slab <= SL_LDS)
        waves *= 2;
    return launch_in_pieces(blocks, 64 * waves, [&](unsigned first, dim3 grid) {
        hipLaunchKernelGGL((fp2d_slab_kernel<T, FAN, SW>), grid, dim3(64 * waves), waves * slab, s, g, views,
                           (const T *)img, (T *)sino, groups, first);
    });
}

template <typename T, bool FAN>
hipError_t fp2d_f(const Geom2D &g, const float2 *views, const void *img, void *sino, int batch, hipStream_t s)
{
    // Slabs, once the waves of rays fill the GPU with as many slabs each as the
    // image is narrow (direct and in slabs, us: 256^2, 180 and 720 waves of rays, 16
    // and 20, 44 and 26; 128^2, 520 and 1300 waves 19.7 and 19.0, 40 and 24; 64^2, 800
    // and 1300 waves 16.7 and 17.2, 24.3 and 18.8; 512 x 64, 800 and 1300 waves 28 and
    // 29, 39 and 35; 121 x 36, 1300 and 2500 waves 13.9 and 16.7, 21.9 and 21.0; below
    // 32 pixels 89 x 26, 5000 waves 27 and 36) and 64 of them fit a slab: the
    // pixels they span along a plane of the walk, at most, are their spacing at
    // the far side of the image, seen along the plane, and the plane's own advance
    // and margins.
    const float wx = g.nx * g.sx, wy = g.ny * g.sy;
    const float far = FAN ? (g.sid + 0.5f * sqrtf(wx * wx + wy * wy)) / g.ru : g.du;
    const float span = 63.0f * 1.4143f * far / fminf(g.sx, g.sy) + SL_D + 5.0f;
    // A wave with few rays walks its slabs all the same: at least half of the
    // lanes have one (256^2 and 40000 rays of 1, 9, 25, 33, 45, 65 and 96 bins: 51
    // us direct at all, in slabs 626, 88, 44, 36, 32, 41 and 40; 700^2: 87 direct,
    // 1700, 220, 140, 108, 91, 122 and 119).
    const long groups = (g.nu + 63) / 64, rays = groups * g.n_proj * batch;   // in waves
    const int narrow = g.nx < g.ny ? g.nx : g.ny;
    if (rays >= 512 && rays * narrow >= 64000 && narrow >= 32 && 2L * g.nu > 64 * groups &&
        g.step <= fminf(g.sx, g.sy)) {
        if (span <= 104.0f)
            return fp2d_slab<T, FAN, 104>(g, views, img, sino, batch, s);
        if (span <= 168.0f)
            return fp2d_slab<T, FAN, 168>(g, views, img, sino, batch, s);
    }
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

template <typename T, typename TI, bool FAN, int NB, int W>
hipError_t bp2d_seg(const Geom2D &g, const float2 *views, const void *sino, void *img, int batch, hipStream_t s)
{
    const int ntx = (g.nx + 15) / 16, nty = (g.ny + 15) / 16;
    const long tiles = (long)ntx * nty * ((batch + NB - 1) / NB);
    // waves per tile: about 32 on every CU in all (8 x 256^2, 360 parallel views
    // one item at a time, in the step of learning the filter: 438, 416 and 418
    // us for 4096, 8192 and 16384), a chunk of views each
    int waves = 1;
    while (waves < 8 && tiles * waves < 8192 && (2 * waves - 1) * (SB_BINS / W) < g.n_proj)
        waves *= 2;
    return launch_in_pieces(tiles, 64 * waves, [&](unsigned first, dim3 grid) {
        hipLaunchKernelGGL((bp2d_seg_kernel<T, TI, FAN, NB, W>), grid, dim3(64 * waves),
                           (size_t)waves * SB_BINS * NB * sizeof(float), s, g, views, (const TI *)sino, (T *)img, ntx,
                           nty, batch, first);
    });
}

template <typename T, typename TI, bool FAN, int NB>
hipError_t bp2d_seg_w(float span, const Geom2D &g, const float2 *views, const void *sino, void *img, int batch,
                      hipStream_t s)
{
    return span <= 28.0f ? bp2d_seg<T, TI, FAN, NB, 32>(g, views, sino, img, batch, s)
                         : bp2d_seg<T, TI, FAN, NB, 64>(g, views, sino, img, batch, s);
}

template <typename T, typename TI, bool FAN>
hipError_t bp2d_f(const Geom2D &g, const float2 *views, const void *sino, void *img, int batch, hipStream_t s)
{
    // From staged bins where those of a 16 x 16 tile, at most its diagonal seen
    // from the near side of the image, fit 64 with the margins.  Items of a
    // batch go together as long as 256 workgroups are left (180 fan views of
    // 128^2: 20, 22 us for one and two together of 2 items, with the filter).
    // Parallel views gain from the staging alone, once there are tiles for most
    // CUs and work to outweigh it (one item, us from memory and staged: 64^2, 90
    // views 4.4 and 9.4, 168^2, 300 views 10 and 13, 200^2, 300 views 13.0 and 13.1,
    // 236^2, 246 views 15.1 and 11.8 with the call, 256^2, 30, 90 and 180 views
    // 4.6 and 6.0, 9.2 and 9.6, 12.1 and 9.9, 320^2, 90 views 13.9 and 10.5, 512^2,
    // 30 and 300 views 9.5 and 6.7, 46.7 and 31.2); fan views, bound by the
    // arithmetic of their coordinates, only where two items or more share it
    // (256^2, 180 flat views of one, two and five items: 16, 30 and 63 us from
    // memory, 20 and 35 for two and five staged).
    const float wx = g.nx * g.sx, wy = g.ny * g.sy, near = g.sid - 0.5f * sqrtf(wx * wx + wy * wy);
    const float diag = 15.0f * sqrtf(g.sx * g.sx + g.sy * g.sy);
    const float span = !FAN ? diag * g.ru : near > 0.0f ? diag * g.ru / near : 3.0e38f;
    const long pieces = (long)((g.nx + 15) / 16) * ((g.ny + 15) / 16);
    int nb = 1;
    while (nb < 4 && nb < batch && pieces * ((batch + 2 * nb - 1) / (2 * nb)) >= 256)
        nb *= 2;
    const long work = pieces * batch;   // tiles
    if (span <= 60.0f && (FAN || (work >= 200 && work * g.n_proj >= 30000))) {
        if (nb == 4)
            return bp2d_seg_w<T, TI, FAN, 4>(span, g, views, sino, img, batch, s);
        if (nb == 2)
            return bp2d_seg_w<T, TI, FAN, 2>(span, g, views, sino, img, batch, s);
        if constexpr (!FAN)
            return bp2d_seg_w<T, TI, FAN, 1>(span, g, views, sino, img, batch, s);
    }
    const int ntx = (g.nx + 7) / 8, nty = (g.ny + 7) / 8;
    const long tiles = (long)ntx * nty * batch;
    // waves per tile: at least 64 per CU in all (512^2, 360 fan views with the
    // filter: 107, 89, 86 and 89 us for 16, 32, 64 and 128), four views each
    int waves = 1;
    while (waves < 16 && tiles * waves < 16384 && 8 * waves <= g.n_proj)
        waves *= 2;
    return launch_in_pieces(tiles, 64 * waves, [&](unsigned first, dim3 grid) {
        hipLaunchKernelGGL((bp2d_kernel<T, TI, FAN>), grid, dim3(64 * waves), waves > 1 ? 64 * waves * sizeof(float) : 0,
                           s, g, views, (const TI *)sino, (T *)img, ntx, nty, first);
    });
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
