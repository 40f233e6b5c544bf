// Device helpers shared by the projector, back-projector and adjoint kernels.
#pragma once

#include "common.h"
#include "fp64.h"

namespace ph {

// Two neighbouring elements in one load (the pair is aligned like its element).
template <typename T>
__device__ __forceinline__ float2 load_pair(const T *base, unsigned bytes)
{
    struct Pair {
        T a, b;
    } p;
    __builtin_memcpy(&p, (const char *)base + (size_t)bytes, sizeof p);
    return make_float2(load_f32(&p.a), load_f32(&p.b));
}

// Orders a wave's own LDS writes before its lanes' reads (and the other way
// round): for LDS that only one wave uses.
__device__ __forceinline__ void wave_lds_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Index coordinates (x, y, z) of a ray's anchor (its point closest to the
// isocentre) and of one sampling step: sample m sits at p + m * e.
struct Ray {
    float p[3], e[3];
};

// 1 / sqrt(x) from the hardware estimate refined by two Newton steps
__device__ __forceinline__ double rsqrt_nr(double x)
{
    const double h = 0.5 * x;
    double r = __builtin_amdgcn_rsq(x);
    r = r * fma(-h * r, r, 1.5);
    return r * fma(-h * r, r, 1.5);
}

// Ray of cone-beam detector pixel (j, i), set up in double precision (the
// source is ~SID away, so an FP32 direction would misplace the ray by
// ~SID * 2^-24 at the volume) and rounded once to FP32.  The direction is
// normalised with the hardware reciprocal square root refined by two Newton
// steps, and the per-view reciprocals of the spacing replace divisions, so
// the set-up takes a few dozen double-precision operations.  The forward
// projector and its transpose both use this, so they see the same samples.
__device__ __forceinline__ Ray make_cone_ray(const Geom3D &g, const ConeFPView &v, int j, int i)
{
    const double jc = (double)j - (double)g.cu, ic = (double)i - (double)g.cv;
    double d[3];
#pragma unroll
    for (int t = 0; t < 3; ++t)
        d[t] = fma(jc, v.du[t], fma(ic, v.dv[t], v.d0[t]));
    const double rn = rsqrt_nr(fma(d[0], d[0], fma(d[1], d[1], d[2] * d[2])));
#pragma unroll
    for (int t = 0; t < 3; ++t)
        d[t] *= rn;
    const double t0 = -(v.s[0] * d[0] + v.s[1] * d[1] + v.s[2] * d[2]);
    const double o[3] = {g.ox, g.oy, g.oz};
    Ray r;
#pragma unroll
    for (int t = 0; t < 3; ++t) {
        r.p[t] = (float)((fma(t0, d[t], v.s[t]) - o[t]) * v.inv_sp[t]);
        r.e[t] = (float)(d[t] * v.step_sp[t]);
    }
    return r;
}

// Sample positions of cone rays are evaluated around a +4 bias on every axis
// (biased coordinates stay positive, so the slab walk can floor by
// truncation); un-biasing is exact (subtracting 4 from a float in [4, 2^20)).
// Every kernel that visits cone samples uses this one expression, so the
// projector and its transpose see bitwise the same positions.
constexpr float RAY_BIAS = 4.0f;

__device__ __forceinline__ float ray_coord_biased(float p_biased, float e, int m)
{
    return fmaf((float)m, e, p_biased);
}

// Ray of 2D detector bin j in a view with central ray vector c: index
// coordinates (x, y) of its anchor and of one step (fan rays set up in double
// precision for the same reason as cone rays).  On the equiangular detector
// bin j sits at fan angle u / SDD on the arc of radius SDD about the source,
// so its ray is the central ray turned by that angle.
template <bool FAN>
__device__ __forceinline__ void make_ray_2d(const Geom2D &g, float2 c, int j, float &X0, float &Y0, float &eX,
                                            float &eY)
{
    const double cx = c.x, cy = c.y, ex = -cy, ey = cx;
    const double u = ((double)j - (double)g.cu) * (double)g.du;
    double ax, ay, dx, dy;
    if (!FAN) {
        ax = u * ex;
        ay = u * ey;
        dx = cx;
        dy = cy;
    } else {
        const double sx = -(double)g.sid * cx, sy = -(double)g.sid * cy;
        if (g.curved) {
            double cg, sg;
            sincos(u / (double)g.sdd, &sg, &cg);
            dx = fma(cg, cx, sg * ex);
            dy = fma(cg, cy, sg * ey);
        } else {
            const double tx = fma((double)g.sdd, cx, u * ex), ty = fma((double)g.sdd, cy, u * ey);  // detector - source
            const double rn = rsqrt64(fma(tx, tx, ty * ty));
            dx = tx * rn;
            dy = ty * rn;
        }
        const double t0 = -fma(sx, dx, sy * dy);
        ax = fma(t0, dx, sx);
        ay = fma(t0, dy, sy);
    }
    X0 = (float)div64(ax - (double)g.ox, (double)g.sx, g.inv_sx);
    Y0 = (float)div64(ay - (double)g.oy, (double)g.sy, g.inv_sy);
    eX = (float)(dx * g.step_sx);
    eY = (float)(dy * g.step_sy);
}

// 1/x from the hardware estimate refined by one Newton step: the correctly
// rounded quotient at every one of the 2^23 mantissas, and so is div_nr's (tried
// with three numerators)
__device__ __forceinline__ float rcp_nr(float x)
{
    const float r = __builtin_amdgcn_rcpf(x);
    return fmaf(r, fmaf(-x, r, 1.0f), r);
}

// n / d from rcp_nr with one more residual step, in five instructions
__device__ __forceinline__ float div_nr(float n, float d)
{
    const float r = rcp_nr(d), q = n * r;
    return fmaf(fmaf(-q, d, n), r, q);
}

// atan(z) / z - 1 = s Q(s), s = z^2, for |z| <= tan(pi / 8): Q interpolated at
// six Chebyshev nodes of [0, tan^2(pi / 8)] (worst error of s Q 1.6e-9).
__device__ __forceinline__ float atan_small(float z)
{
    const float s = z * z;
    float q = fmaf(s, 0.050471332f, -0.08624286f);
    q = fmaf(s, q, 0.110713124f);
    q = fmaf(s, q, -0.14284149f);
    q = fmaf(s, q, 0.19999978f);
    q = fmaf(s, q, -0.33333334f);
    return fmaf(z * s, q, z);
}

// Bin fu (a float whole number), fraction t and distance weight wt of world
// point (x, y) in a 2D view with central ray c.  Parallel beams: the
// orthogonal projection, weight 1.  Fan beams: central projection onto the
// flat detector with weight (SID / w)^2, w the depth along the central ray; on
// the equiangular detector the bin of the point's fan angle, with weight
// (SID / L)^2, L the distance from the source.  All in FP32.
//
// B and B^T take every coordinate from here and so see the same ones to the
// last bit, on every detector.  FORM names the detector, so that the code has
// no branch on it.  Arcs of few bins (FORM_FINE_ARC, ru_lo not 0): the fan
// angle is atan_small of the slope, taken from the pi / 4 or pi / 2 direction
// beyond tan(pi / 8) and tan(3 pi / 8) (where no lane of the wave is beyond, or
// FORM_SMALL says so, that is left out: the same value, every step is odd in
// xu); the scale to bins is held in two floats and the fraction is formed from
// the centred coordinate, since there the rounding of their sum would be the
// largest error.  On longer arcs (FORM_ARC) the fan angle is atan2f's: whatever
// its own error, the sum rounds to 2^-15 bin at 512 to 1023 bins, and results
// for rough data are only as reproducible as its last bits.
//
// FORM_RANGE, for ranges of bins with a margin of more than 1e-3 bin: the
// polynomial on every arc, whichever detector it is.
constexpr int FORM_FLAT = 1, FORM_FINE_ARC = 2, FORM_ARC = 4, FORM_SMALL = 8, FORM_RANGE = 16;

template <bool FAN, int FORM>
__device__ __forceinline__ void point2d(const Geom2D &g, float2 c, float x, float y, float &fu, float &t, float &wt)
{
#pragma clang fp contract(off)   // the fused operations are those written out, in every caller
    const float xu = fmaf(y, c.x, -(x * c.y));
    float s;   // detector coordinate in bins
    wt = 1.0f;
    if (!FAN) {
        s = fmaf(xu, g.ru, g.cu);
    } else {
        const float w = fmaf(x, c.x, fmaf(y, c.y, g.sid));
        if (FORM == FORM_FLAT || (FORM == FORM_RANGE && !g.curved)) {
            const float rw = rcp_nr(w), sw = g.sid * rw;
            s = fmaf(g.sdd * xu * rw, g.rdu, g.cu);
            wt = sw * sw;
        } else {
            wt = div_nr(g.sid * g.sid, fmaf(w, w, xu * xu));
            if (FORM == FORM_ARC) {
                // the clamps change nothing for a point in front of the source; they
                // tell the compiler which of atan2f's special cases cannot occur
                // (nine of its operations)
                const float xc = fminf(fmaxf(xu, -1e30f), 1e30f), wc = fminf(fmaxf(w, 1e-30f), 1e30f);
                s = fmaf(atan2f(xc, wc), g.ru, g.cu);
            } else {
                const float a = fabsf(xu);
                float q, off = 0.0f;   // fan angle: q + off
                if (!(FORM & FORM_SMALL) && __any(a > 0.41421357f * w)) {
                    float num = a, den = w;
                    if (a > 0.41421357f * w) {
                        const bool steep = a > 2.4142135f * w;
                        num = steep ? -w : a - w;
                        den = steep ? a : a + w;
                        off = copysignf(steep ? 1.57079633f : 0.78539816f, xu);
                    }
                    q = copysignf(1.0f, xu) * atan_small(div_nr(num, den));
                } else {
                    q = atan_small(div_nr(xu, w));
                }
                if (FORM != FORM_RANGE) {
                    const float lo = (q + off) * g.ru_lo;
                    fu = floorf(fmaf(q, g.ru, fmaf(off, g.ru, g.cu) + lo));
                    t = fmaf(q, g.ru, fmaf(off, g.ru, g.cu - fu)) + lo;
                    return;
                }
                s = fmaf(q + off, g.ru, g.cu);
            }
        }
    }
    fu = floorf(s);
    t = s - fu;
}

template <int F>
struct Form {   // a form of point2d as an argument
    static constexpr int value = F;
};

// use(Form<...>()) with the form of g's detector (uniform branches)
template <bool FAN, typename Use>
__device__ __forceinline__ void with_form(const Geom2D &g, Use use)
{
    if (!FAN || !g.curved)
        use(Form<FORM_FLAT>());
    else if (g.ru_lo != 0.0f)
        use(Form<FORM_FINE_ARC>());
    else
        use(Form<FORM_ARC>());
}

// Narrow [lo, hi] to the parameters t with p + t e inside the open interval
// (a, b); false if the line never enters it.
__device__ __forceinline__ bool clip_line(float p, float e, float a, float b, float &lo, float &hi)
{
    if (fabsf(e) < 1e-30f)
        return p > a && p < b;
    const float t1 = (a - p) / e, t2 = (b - p) / e;
    lo = fmaxf(lo, fminf(t1, t2));
    hi = fminf(hi, fmaxf(t1, t2));
    return true;
}

// clip_line with the hardware reciprocal in place of the divisions: the
// bounds may be off by a few ulps, so callers widen the range they derive and
// test each sample exactly.
__device__ __forceinline__ bool clip_line_rcp(float p, float e, float a, float b, float &lo, float &hi)
{
    if (fabsf(e) < 1e-30f)
        return p > a && p < b;
    const float r = __builtin_amdgcn_rcpf(e);
    const float t1 = (a - p) * r, t2 = (b - p) * r;
    lo = fmaxf(lo, fminf(t1, t2));
    hi = fminf(hi, fmaxf(t1, t2));
    return true;
}

__device__ __forceinline__ float dot4(const float r[4], float x, float y, float z)
{
    return fmaf(r[0], x, fmaf(r[1], y, fmaf(r[2], z, r[3])));
}

// nearest integer of x (ties toward +inf) in one instruction; the
// fixed-point LDS accumulators of the transposes round every term with it
__device__ __forceinline__ int round_to_int(float x)
{
    int r;
    asm("v_cvt_rpi_i32_f32 %0, %1" : "=v"(r) : "v"(x));
    return r;
}

template <int CTRL>
__device__ __forceinline__ float dpp(float x)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, false));
}

// min / max over the 8 corners held by lanes with corner index lane mod 8:
// xor 1 and xor 2 within quads, then rotate each 16-lane row by 4 lanes,
// which pairs a quad holding corners 0-3 with one holding corners 4-7.
__device__ __forceinline__ float min8(float x)
{
    x = fminf(x, dpp<0xB1>(x));
    x = fminf(x, dpp<0x4E>(x));
    return fminf(x, dpp<0x124>(x));
}
__device__ __forceinline__ float max8(float x)
{
    x = fmaxf(x, dpp<0xB1>(x));
    x = fmaxf(x, dpp<0x4E>(x));
    return fmaxf(x, dpp<0x124>(x));
}

// the same over integers (no NaN handling, so each step is one DPP min/max)
template <int CTRL>
__device__ __forceinline__ int dppi(int x)
{
    return __builtin_amdgcn_update_dpp(0, x, CTRL, 0xF, 0xF, false);
}
__device__ __forceinline__ int imin4(int x)   // over four corners, lane mod 4
{
    x = min(x, dppi<0xB1>(x));
    return min(x, dppi<0x4E>(x));
}
__device__ __forceinline__ int imax4(int x)
{
    x = max(x, dppi<0xB1>(x));
    return max(x, dppi<0x4E>(x));
}
__device__ __forceinline__ int imin8(int x)
{
    x = min(x, dppi<0xB1>(x));
    x = min(x, dppi<0x4E>(x));
    return min(x, dppi<0x124>(x));
}
__device__ __forceinline__ int imax8(int x)
{
    x = max(x, dppi<0xB1>(x));
    x = max(x, dppi<0x4E>(x));
    return max(x, dppi<0x124>(x));
}

}  // namespace ph
