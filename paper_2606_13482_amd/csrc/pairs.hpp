// Kernel sums of one triangle pair (device code shared by the fill, the near
// entries of the fast operator and the Calderon preconditioner's dual matrix).
//
// On triangles p and q, with points x_i, y_j relative to the centroids c_p, c_q
// and d = c_p - c_q, the local blocks of the operator need
//     S0 = sum_ij w_i w_j g_ij,   Sx = sum w_i w_j g_ij x_i,   Sy = sum w_i w_j g_ij y_j,
//     Sxy = sum w_i w_j g_ij (x_i . y_j),   g_ij = exp(-jk R_ij) / (4 pi R_ij),
//     R_ij = |d + x_i - y_j|.
//
// These 49 kernel values bound the FP64 fill (FP64 vector issue).  exp(-jk R_ij)
// is exp(-jk |d|) exp(-j k (R_ij - |d|)): the first factor is common to the pair
// and multiplies the sums at the end, and the second has a small argument, at
// most k times the two triangles' point radii (0.5 at ten edges per wavelength),
// so sine and cosine are two short polynomials with no argument reduction and
// no selection.  A pair whose bound exceeds NARROW_PHASE takes the library's
// sincos.  With the reciprocal root from v_rsq_f64 and one third-order
// correction a kernel value takes about 50 FP64 instructions; 1 / sqrt and
// sincos took about 180.
#pragma once

#include "bie_internal.hpp"

namespace bie {

// largest |k (R_ij - |d|)| of the polynomials below
constexpr double NARROW_PHASE = 1.3;

// sin t and cos t for |t| <= NARROW_PHASE: interpolation of sin(sqrt u)/sqrt u and
// cos(sqrt u) at the Chebyshev points of u in [0, NARROW_PHASE^2], evaluated in 60
// digits (error of the polynomials 1.6e-17 and 1.5e-17; the leading ones are 1).
__device__ __forceinline__ void sincos_narrow(double t, double &s, double &c)
{
    const double u = t * t;
    double a = -7.45932327614400113e-13, b = 4.66206985662428132e-14;
    a = __builtin_fma(a, u, 1.60539051356314017e-10);
    b = __builtin_fma(b, u, -1.14670395521753741e-11);
    a = __builtin_fma(a, u, -2.50520350393927523e-08);
    b = __builtin_fma(b, u, 2.08766937788810224e-09);
    a = __builtin_fma(a, u, 2.75573186435645317e-06);
    b = __builtin_fma(b, u, -2.75573185951748121e-07);
    a = __builtin_fma(a, u, -1.98412698387745771e-04);
    b = __builtin_fma(b, u, 2.48015872979112463e-05);
    a = __builtin_fma(a, u, 8.33333333332806486e-03);
    b = __builtin_fma(b, u, -1.38888888888768136e-03);
    a = __builtin_fma(a, u, -1.66666666666666241e-01);
    b = __builtin_fma(b, u, 4.16666666666664701e-02);
    b = __builtin_fma(b, u, -0.5);
    s = __builtin_fma(t * u, a, t);
    c = __builtin_fma(b, u, 1.0);
}

// sin t and cos t: t less its nearest multiple n of pi/2 is in the narrow range.
// pi/2 in three parts (Cody and Waite 1980; the first two of 33 bits, so that
// their products with n are exact); beyond |t| = 1e5 the library's reduction.
__device__ __forceinline__ void sincos_reduced(double t, double &s, double &c)
{
    if (!(fabs(t) <= 1e5)) {
        sincos(t, &s, &c);
        return;
    }
    const double n = rint(t * 0.63661977236758134308);
    double r = __builtin_fma(-n, 0x1.921fb54400000p+0, t);
    r = __builtin_fma(-n, 0x1.0b4611a600000p-34, r);
    r = __builtin_fma(-n, 0x1.3198a2e037073p-69, r);
    double a, b;
    sincos_narrow(r, a, b);
    const int q = int(n);
    s = (q & 1) ? b : a;
    c = (q & 1) ? a : b;
    if (q & 2) s = -s;
    if ((q + 1) & 2) c = -c;
}

// 1 / sqrt(x): the hardware estimate (relative error e below 2^-20) and the
// expansion (1 - e)^(-1/2) = 1 + e/2 + 3 e^2/8 of its error
__device__ __forceinline__ double rsqrt_fast(double x)
{
    const double y = __builtin_amdgcn_rsq(x);
    const double e = __builtin_fma(-(x * y), y, 1.0);
    return __builtin_fma(y * e, __builtin_fma(e, 0.375, 0.5), y);
}

template <typename R>
struct PairSums {
    R s0r, s0i, sxr[3], sxi[3], syr[3], syi[3], sxyr, sxyi;
};

template <typename R>
__device__ __forceinline__ void sincos_any(R x, R &s, R &c);
template <>
__device__ __forceinline__ void sincos_any<double>(double x, double &s, double &c) { sincos_reduced(x, s, c); }
template <>
__device__ __forceinline__ void sincos_any<float>(float x, float &s, float &c)
{
    // Reduce to [-1/2, 1/2] revolutions, then the hardware sine / cosine.
    const float rev = x * 0.15915494309189533577f;
    const float f = rev - rintf(rev);
    s = __builtin_amdgcn_sinf(f);
    c = __builtin_amdgcn_cosf(f);
}
__device__ __forceinline__ double rsqrt_any(double x) { return rsqrt_fast(x); }
__device__ __forceinline__ float rsqrt_any(float x) { return rsqrtf(x); }

// x: the 7 points of p (the same for every lane), y: those of q, w: the rule's
// weights, w4: weights / (4 pi).  NARROW (double only): k (R - |d|) is at most
// NARROW_PHASE for every point pair.
// y is called as y(j, c).
template <typename R, bool NARROW, typename Y>
__device__ __forceinline__ void pair_sums(const R *__restrict__ x, const Y &yq, const R (&d)[3], R k,
                                          const R *__restrict__ w, const R *__restrict__ w4, PairSums<R> &S)
{
    R r0 = 0;
    if (NARROW) r0 = sqrt(d[0] * d[0] + d[1] * d[1] + d[2] * d[2]);
    S.s0r = S.s0i = S.sxyr = S.sxyi = 0;
#pragma unroll
    for (int c = 0; c < 3; ++c) S.sxr[c] = S.sxi[c] = S.syr[c] = S.syi[c] = 0;
#pragma unroll 1
    for (int i = 0; i < QPTS; ++i) {
        const R xi[3] = { x[3 * i], x[3 * i + 1], x[3 * i + 2] };
        const R di[3] = { d[0] + xi[0], d[1] + xi[1], d[2] + xi[2] };
        R tr = 0, ti = 0, yr[3] = { 0, 0, 0 }, yi[3] = { 0, 0, 0 };
#pragma unroll
        for (int j = 0; j < QPTS; ++j) {
            const R y[3] = { yq(j, 0), yq(j, 1), yq(j, 2) };
            const R e0 = di[0] - y[0], e1 = di[1] - y[1], e2 = di[2] - y[2];
            const R r2 = e0 * e0 + e1 * e1 + e2 * e2;
            const R ri = rsqrt_any(r2);
            R sn, cs;
            if constexpr (NARROW) sincos_narrow(k * (r2 * ri - r0), sn, cs);
            else sincos_any<R>(k * (r2 * ri), sn, cs);
            const R gw = w4[j] * ri;
            const R gr = gw * cs, gi = -gw * sn;
            tr += gr;
            ti += gi;
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                yr[c] += gr * y[c];
                yi[c] += gi * y[c];
            }
        }
        const R a = w[i];
        const R atr = a * tr, ati = a * ti;
        S.s0r += atr;
        S.s0i += ati;
        R xr = 0, xm = 0;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            S.sxr[c] += atr * xi[c];
            S.sxi[c] += ati * xi[c];
            S.syr[c] += a * yr[c];
            S.syi[c] += a * yi[c];
            xr += xi[c] * yr[c];
            xm += xi[c] * yi[c];
        }
        S.sxyr += a * xr;
        S.sxyi += a * xm;
    }
    if (NARROW) {   // the common factor exp(-jk |d|)
        R sn, cs;
        sincos_any<R>(k * r0, sn, cs);
        auto turn = [&](R &re, R &im) {
            const R t = re * cs + im * sn;
            im = im * cs - re * sn;
            re = t;
        };
        turn(S.s0r, S.s0i);
        turn(S.sxyr, S.sxyi);
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            turn(S.sxr[c], S.sxi[c]);
            turn(S.syr[c], S.syi[c]);
        }
    }
}

// L_ab = s_a s_b [ (jk/4) J_ab + S0/(jk) ] with J_ab = Sxy - v_b.Sx - v_a.Sy + (v_a.v_b) S0
// (v relative to the own centroid), or with SPLIT only the J_ab part: row a, b = 0..2.
template <typename R, bool SPLIT>
__device__ __forceinline__ void local_row(const PairSums<R> &S, const R (&va)[3], const R (&vb)[3][3], R sa,
                                          const R (&sb)[3], R k4, R ik, R (&lr)[3], R (&li)[3])
{
    R ar = S.sxyr, ai = S.sxyi;
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        ar -= va[c] * S.syr[c];
        ai -= va[c] * S.syi[c];
    }
#pragma unroll
    for (int b = 0; b < 3; ++b) {
        const R vv = va[0] * vb[b][0] + va[1] * vb[b][1] + va[2] * vb[b][2];
        R jr = ar + vv * S.s0r, ji = ai + vv * S.s0i;
#pragma unroll
        for (int c = 0; c < 3; ++c) {
            jr -= vb[b][c] * S.sxr[c];
            ji -= vb[b][c] * S.sxi[c];
        }
        const R ss = sa * sb[b];
        lr[b] = SPLIT ? ss * (-k4 * ji) : ss * (-k4 * ji + ik * S.s0i);
        li[b] = SPLIT ? ss * (k4 * jr) : ss * (k4 * jr - ik * S.s0r);
    }
}

}  // namespace bie
