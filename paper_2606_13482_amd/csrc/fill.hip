// Dense EFIE impedance matrix fill, plane-wave excitation and radiation vector.
//
// Operator (Sec. II, eq:efie, eq:matTA, eq:matTPhi) in RWG functions without
// edge-length normalisation.  On triangle p of f_m: f_m = s (r - v)/(2 A_p),
// div f_m = s / A_p.  For a triangle pair (p, q) and local slots a, b the
// contribution to T_{m(p,a), n(q,b)} is
//     L_ab = s_a s_b [ (jk/4) J_ab + J0/(jk) ],
//     J_ab = sum_ij w_i w_j (x_i - v_a).(y_j - v_b) g(|x_i - y_j|),  J0 = sum_ij w_i w_j g
// with area-relative weights (the areas cancel against 1/(A_p A_q)).  The
// minus signs of eq:efie and eq:matTPhi cancel.
//
// Star-split form (Sec. VI-A, star factorisation of the scalar potential):
// with div f_m = +-1/A on c_m^+- the scalar term of T is Sigma V Sigma^T,
// Sigma_mp = s (the sign of triangle p in RWG m) and V_pq = J0 / (jk) the
// piecewise-constant single layer (basis 1/A) scaled by 1/(jk).  In that form
// the local blocks keep only the vector part s_a s_b (jk/4) J_ab (assembled
// into T_A' = jk T_A exactly as T), and J0 / (jk) of every pair p <= q is
// written to its own tile array and assembled into packed F x F tiles of V'.
//
// Pipeline (three launches, no atomics, bitwise symmetric result):
//   1. k_pairs_regular: one lane per triangle pair p <= q; 49 kernel evaluations;
//      writes the 3x3 local block L into a scratch array of bands of 16 rows p.
//   2. k_pairs_singular: 16 lanes per flagged pair (touching or near), FP64:
//      g = g_r + 1/(4 pi R), g_r on the product rule, the static part with the
//      inner integral in closed form, mean of both orderings; overwrites L.
//   3. k_assemble: T_mn = (L(c+m,c+n) + L(c-m,c-n)) + (L(c+m,c-n) + L(c-m,c+n));
//      the grouping makes T_mn and T_nm the same sum, so T = T^T exactly, and
//      only the upper-triangular 64 x 64 tiles are written (packed storage).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <type_traits>
#include <vector>

#include "bie_internal.hpp"
#include "pairs.hpp"

namespace bie {

namespace {

constexpr int TT = 16;               // rows of a band of the pair scratch
constexpr int NQ = 7;                // Radon 7-point rule
constexpr double PI = 3.14159265358979323846;

// Radon's degree-5 rule: centroid, orbits (a,a,1-2a) with a = (6 -+ sqrt(15))/21.
struct Rule {
    double bary[NQ][3];
    double w[NQ];
};

Rule make_rule()
{
    Rule r;
    const double s = std::sqrt(15.0);
    const double a = (6.0 - s) / 21.0, b = (6.0 + s) / 21.0;
    const double wa = (155.0 - s) / 1200.0, wb = (155.0 + s) / 1200.0;
    const double pts[NQ][3] = { { 1.0 / 3, 1.0 / 3, 1.0 / 3 },
                                { a, a, 1 - 2 * a }, { a, 1 - 2 * a, a }, { 1 - 2 * a, a, a },
                                { b, b, 1 - 2 * b }, { b, 1 - 2 * b, b }, { 1 - 2 * b, b, b } };
    const double ws[NQ] = { 9.0 / 40.0, wa, wa, wa, wb, wb, wb };
    for (int i = 0; i < NQ; ++i) {
        for (int d = 0; d < 3; ++d) r.bary[i][d] = pts[i][d];
        r.w[i] = ws[i];
    }
    return r;
}

// the rule's weights: 9/40, three times (155 - sqrt 15)/1200, three times (155 + sqrt 15)/1200
__constant__ double c_w[NQ] = { 0.225, 0x1.01ec66adccf2ap-3, 0x1.01ec66adccf2ap-3, 0x1.01ec66adccf2ap-3,
                                0x1.0f24aa63441e7p-3, 0x1.0f24aa63441e7p-3, 0x1.0f24aa63441e7p-3 };

// Scratch of the local blocks: triangles in the device order, in bands of TT
// rows p; band I holds the columns q >= TT I up to Fp (F rounded up to TT) and
// its rows are [slot a of p][q][slot b of q].  Lanes over q write whole lines, and
// the assembly, which walks the functions n of one row m, finds the three slots
// of a triangle q side by side.
struct Bands {
    int64_t Fp;
    __host__ __device__ int64_t cols(int64_t I) const { return Fp - TT * I; }
    __host__ __device__ int64_t base(int64_t I) const { return TT * (I * Fp - TT * (I * (I - 1) / 2)); }   // pairs before band I
    __host__ __device__ int64_t total() const { return base(Fp / TT); }
    // complex entry of slots (a, b) of the pair p <= q
    __device__ int64_t block(int64_t p, int64_t q, int a, int b) const
    {
        const int64_t I = p / TT;
        return 9 * base(I) + (((p % TT) * 3 + a) * cols(I) + (q - TT * I)) * 3 + b;
    }
    __device__ int64_t pair(int64_t p, int64_t q) const
    {
        const int64_t I = p / TT;
        return base(I) + (p % TT) * cols(I) + (q - TT * I);
    }
};

// ---------------------------------------------------------------------------
// 1. Regular pairs.  A lane keeps one triangle q in registers and goes through
// the triangles p of a band, which LDS hands to all lanes at once; the sums
// of a pair are pairs.hpp's.  In FP64 the pairs beyond NARROW_PHASE are left to a
// launch of their own (NARROW false), made only if the mesh can have any: in one
// kernel with them the narrow form has two waves per SIMD instead of three.  A
// block takes the band's rows p = blockIdx.z, blockIdx.z + gridDim.z, ...  FP64 vector issue bounds it: 13.1 M pairs
// (7680 unknowns) 2.92 -> 1.50 ms, 54 vector instructions a kernel value, the vector
// units busy 73 % of the time at 2.0 GHz; three waves per SIMD instead of two (y in
// LDS) measured the same.
template <typename R, bool SPLIT, bool NARROW>
__global__ __launch_bounds__(256) void k_pairs_regular(int64_t F, Bands bd, const double *__restrict__ cent,
                                                       const double *__restrict__ loc,
                                                       const double *__restrict__ vfree,
                                                       const int8_t *__restrict__ sgn,
                                                       const double *__restrict__ rad, double k,
                                                       R *__restrict__ LB, R *__restrict__ VS)
{
    __shared__ R sx[TT][NQ * 3], sv[TT][9], ss[TT][3];
    __shared__ double sc[TT][3], sr[TT];
    __shared__ R sw[NQ], sw4[NQ];   // w and w / (4 pi)
    const int64_t I = blockIdx.y, q0 = I * TT + int64_t(blockIdx.x) * 256;
    if (q0 >= F) return;
    const int tid = threadIdx.x;
    for (int e = tid; e < TT * (NQ * 3 + 9 + 3 + 3 + 1); e += 256) {
        const int t = e / (NQ * 3 + 16), f = e % (NQ * 3 + 16);
        const int64_t tri = I * TT + t;
        const bool in = tri < F;
        if (f < NQ * 3) sx[t][f] = in ? R(loc[tri * NQ * 3 + f]) : R(0);
        else if (f < NQ * 3 + 9) sv[t][f - NQ * 3] = in ? R(vfree[tri * 9 + f - NQ * 3]) : R(0);
        else if (f < NQ * 3 + 12) ss[t][f - NQ * 3 - 9] = in ? R(sgn[tri * 3 + f - NQ * 3 - 9]) : R(0);
        else if (f < NQ * 3 + 15) sc[t][f - NQ * 3 - 12] = in ? cent[tri * 3 + f - NQ * 3 - 12] : 0.0;
        else sr[t] = in ? rad[tri] : 0.0;
    }
    if (tid < NQ) {
        sw[tid] = R(c_w[tid]);
        sw4[tid] = R(c_w[tid] / (4.0 * PI));
    }
    __syncthreads();
    const int64_t q = q0 + tid;
    if (q >= F) return;
    R yq[NQ][3];
#pragma unroll
    for (int j = 0; j < NQ; ++j)
#pragma unroll
        for (int c = 0; c < 3; ++c) yq[j][c] = R(loc[(q * NQ + j) * 3 + c]);
    const auto y = [&](int j, int c) { return yq[j][c]; };
    const double cq[3] = { cent[3 * q], cent[3 * q + 1], cent[3 * q + 2] };
    const double rq = rad[q];
    const R kk = R(k), k4 = kk * R(0.25), ik = R(1.0) / kk;
    const int np = int(q - I * TT + 1 < TT ? q - I * TT + 1 : TT);   // p <= q
#pragma unroll 1
    for (int t = blockIdx.z; t < np; t += gridDim.z) {
        const R d[3] = { R(sc[t][0] - cq[0]), R(sc[t][1] - cq[1]), R(sc[t][2] - cq[2]) };
        PairSums<R> S;
        // FP64: a wave's pairs are one launch's or the other's
        if (sizeof(R) == 8 && (__all(k * (sr[t] + rq) <= NARROW_PHASE) != 0) != NARROW) continue;
        pair_sums<R, NARROW>(sx[t], y, d, kk, sw, sw4, S);
        R vb[3][3], sb[3];
#pragma unroll
        for (int b = 0; b < 3; ++b) {
            sb[b] = R(sgn[q * 3 + b]);
#pragma unroll
            for (int c = 0; c < 3; ++c) vb[b][c] = R(vfree[q * 9 + 3 * b + c]);
        }
        const int64_t p = I * TT + t;
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            const R va[3] = { sv[t][3 * a], sv[t][3 * a + 1], sv[t][3 * a + 2] };
            R lr[3], li[3];
            local_row<R, SPLIT>(S, va, vb, ss[t][a], sb, k4, ik, lr, li);
            R *out = LB + 2 * bd.block(p, q, a, 0);
#pragma unroll
            for (int b = 0; b < 3; ++b) {
                out[2 * b] = lr[b];
                out[2 * b + 1] = li[b];
            }
        }
        if (SPLIT) {   // V'_pq = J0 / (jk)
            R *out = VS + 2 * bd.pair(p, q);
            out[0] = ik * S.s0i;
            out[1] = -ik * S.s0r;
        }
    }
}

// ---------------------------------------------------------------------------
// 2. Flagged pairs, FP64.
//
// K0 = int_tri 1/|y-x|, K1 = int_tri (y-x)/|y-x| in closed form (Wilton et al.
// 1984, Graglia 1993): per edge P->Q (CCW about the unit normal n), with
// h = n.(x-P), rho = x - h n, l = (Q-P)/|Q-P|, u = l x n,
// l+- = (Q|P - rho).l, P0 = (P - rho).u, R0^2 = P0^2 + h^2, R+- = sqrt(R0^2 + l+-^2),
// f = ln((R+ + l+)/(R- + l-)) (or ln((R- - l-)/(R+ - l+)) if l+ + l- < 0),
// beta = atan(P0 l+/(R0^2 + |h| R+)) - atan(P0 l-/(R0^2 + |h| R-)):
//   K0 = sum P0 f - |h| beta,  K1 = 1/2 sum u (R0^2 f + l+ R+ - l- R-) - h n K0.
__device__ void static_potentials(const double x[3], const double A[3], const double B[3],
                                  const double C[3], double *K0, double K1[3])
{
    double e1[3], e2[3], n[3];
    for (int d = 0; d < 3; ++d) { e1[d] = B[d] - A[d]; e2[d] = C[d] - A[d]; }
    n[0] = e1[1] * e2[2] - e1[2] * e2[1];
    n[1] = e1[2] * e2[0] - e1[0] * e2[2];
    n[2] = e1[0] * e2[1] - e1[1] * e2[0];
    const double nn = 1.0 / sqrt(n[0] * n[0] + n[1] * n[1] + n[2] * n[2]);
    n[0] *= nn; n[1] *= nn; n[2] *= nn;
    const double h = (x[0] - A[0]) * n[0] + (x[1] - A[1]) * n[1] + (x[2] - A[2]) * n[2];
    const double ah = fabs(h);
    const double rho[3] = { x[0] - h * n[0], x[1] - h * n[1], x[2] - h * n[2] };
    const double *Ps[3] = { A, B, C }, *Qs[3] = { B, C, A };
    double k0 = 0.0, kp[3] = { 0.0, 0.0, 0.0 };
    for (int e = 0; e < 3; ++e) {
        const double *P = Ps[e], *Q = Qs[e];
        double l[3] = { Q[0] - P[0], Q[1] - P[1], Q[2] - P[2] };
        const double il = 1.0 / sqrt(l[0] * l[0] + l[1] * l[1] + l[2] * l[2]);
        l[0] *= il; l[1] *= il; l[2] *= il;
        const double u[3] = { l[1] * n[2] - l[2] * n[1], l[2] * n[0] - l[0] * n[2], l[0] * n[1] - l[1] * n[0] };
        const double lp = (Q[0] - rho[0]) * l[0] + (Q[1] - rho[1]) * l[1] + (Q[2] - rho[2]) * l[2];
        const double lm = (P[0] - rho[0]) * l[0] + (P[1] - rho[1]) * l[1] + (P[2] - rho[2]) * l[2];
        const double P0 = (P[0] - rho[0]) * u[0] + (P[1] - rho[1]) * u[1] + (P[2] - rho[2]) * u[2];
        const double R0s = P0 * P0 + h * h;
        const double Rp = sqrt(R0s + lp * lp), Rm = sqrt(R0s + lm * lm);
        double f = 0.0;
        if (R0s > 0.0) f = (lp + lm < 0.0) ? log((Rm - lm) / (Rp - lp)) : log((Rp + lp) / (Rm + lm));
        // the two arc tangents lie in (-pi/2, pi/2): their difference is one angle
        double beta = 0.0;
        if (ah > 0.0) {
            const double yp = P0 * lp, xp = R0s + ah * Rp, ym = P0 * lm, xm = R0s + ah * Rm;
            beta = atan2(yp * xm - xp * ym, xp * xm + yp * ym);
        }
        k0 += (R0s > 0.0 ? P0 * f : 0.0) - ah * beta;
        const double c = 0.5 * ((R0s > 0.0 ? R0s * f : 0.0) + lp * Rp - lm * Rm);
        kp[0] += c * u[0]; kp[1] += c * u[1]; kp[2] += c * u[2];
    }
    *K0 = k0;
    for (int d = 0; d < 3; ++d) K1[d] = kp[d] - h * n[d] * k0;
}

// 16 lanes per pair: the 49 point pairs of the regular remainder and the 14
// closed-form outer points are spread over them, each adding to the sums of
// pairs.hpp (the static part, real, has the same form: with A = int 1/R and
// B = int y/R over the inner triangle, (x - v_a).(B - v_b A) at outer point x), then
// 9 lanes form the block.  One lane per pair was a serial chain of 14 closed forms
// (3 logarithms and 6 arc tangents each) at one wave per SIMD (5750 pairs 75 -> 15 us,
// 92 450 pairs 185 -> 130 us).
constexpr int SL = 16;
template <typename R, bool SPLIT>
__global__ __launch_bounds__(256) void k_pairs_singular(int64_t npairs, Bands bd,
                                                        const int32_t *__restrict__ pairs,
                                                        const double *__restrict__ cent,
                                                        const double *__restrict__ loc,
                                                        const double *__restrict__ vfree,
                                                        const double *__restrict__ verts,
                                                        const double *__restrict__ area,
                                                        const int8_t *__restrict__ sgn, double k,
                                                        R *__restrict__ LB, R *__restrict__ VS,
                                                        double *__restrict__ compact = nullptr)
{
    const int l = threadIdx.x & (SL - 1);
    const int64_t at = (int64_t(blockIdx.x) * blockDim.x + threadIdx.x) / SL;
    const bool live = at < npairs;
    const int64_t idx = live ? at : npairs - 1;   // the sums below cross lanes: all take part
    const int64_t p = pairs[2 * idx], q = pairs[2 * idx + 1];
    // frames: p-local coordinates relative to c_p, q-local relative to c_q
    double dc[3];
    for (int d = 0; d < 3; ++d) dc[d] = cent[p * 3 + d] - cent[q * 3 + d];
    const double *xl = loc + p * NQ * 3, *yl = loc + q * NQ * 3;
    const double inv4pi = 1.0 / (4.0 * PI);
    PairSums<double> S;
    S.s0r = S.s0i = S.sxyr = S.sxyi = 0.0;
    for (int c = 0; c < 3; ++c) S.sxr[c] = S.sxi[c] = S.syr[c] = S.syi[c] = 0.0;
    // regular remainder g_r = (e^{-jkR} - 1)/(4 pi R) = -2 sin(kR/2) (sin(kR/2) + j cos(kR/2))/(4 pi R)
    for (int e = l; e < NQ * NQ; e += SL) {
        const int i = e / NQ, j = e % NQ;
        const double *x = xl + 3 * i, *y = yl + 3 * j;
        const double d0 = dc[0] + x[0] - y[0], d1 = dc[1] + x[1] - y[1], d2 = dc[2] + x[2] - y[2];
        const double Rr = sqrt(d0 * d0 + d1 * d1 + d2 * d2);
        double gr = 0.0, gi = -k;
        if (Rr > 0.0) {
            double sn, cs;
            sincos_reduced(0.5 * k * Rr, sn, cs);
            const double h = -2.0 * sn / Rr;
            gr = h * sn;
            gi = h * cs;
        }
        const double w = c_w[i] * c_w[j] * inv4pi;
        gr *= w;
        gi *= w;
        S.s0r += gr;
        S.s0i += gi;
        const double xy = x[0] * y[0] + x[1] * y[1] + x[2] * y[2];
        S.sxyr += gr * xy;
        S.sxyi += gi * xy;
        for (int c = 0; c < 3; ++c) {
            S.sxr[c] += gr * x[c];
            S.sxi[c] += gi * x[c];
            S.syr[c] += gr * y[c];
            S.syi[c] += gi * y[c];
        }
    }
    // static part, real: lanes 0..6 p outer / closed form over q, lanes 7..13 q outer
    // / over p; mean of the two orderings
    if (l < 2 * NQ) {
        const bool po = l < NQ;
        const int i = po ? l : l - NQ;
        const int64_t in = po ? q : p;
        const double *ol = po ? xl + 3 * i : yl + 3 * i;
        double u[3], tri[9];   // the outer point and the inner triangle in the inner frame
        for (int d = 0; d < 3; ++d) {
            u[d] = po ? dc[d] + ol[d] : ol[d] - dc[d];
            for (int v = 0; v < 3; ++v) tri[v * 3 + d] = verts[in * 9 + v * 3 + d] - cent[in * 3 + d];
        }
        double K0, K1[3];
        static_potentials(u, tri, tri + 3, tri + 6, &K0, K1);
        const double f = 0.5 * c_w[i] * inv4pi / area[in];
        const double f0 = f * K0;
        S.s0r += f0;
        for (int c = 0; c < 3; ++c) {
            const double B = f * K1[c] + u[c] * f0, A = f0 * ol[c];
            S.sxyr += ol[c] * B;
            if (po) {
                S.sxr[c] += A;
                S.syr[c] += B;
            } else {
                S.sxr[c] += B;
                S.syr[c] += A;
            }
        }
    }
    auto total = [&](double &v) {
#pragma unroll
        for (int o = SL / 2; o > 0; o >>= 1) v += __shfl_xor(v, o, SL);
    };
    total(S.s0r);
    total(S.s0i);
    total(S.sxyr);
    total(S.sxyi);
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        total(S.sxr[c]);
        total(S.sxi[c]);
        total(S.syr[c]);
        total(S.syi[c]);
    }
    if (!live || l >= 9) return;
    const double k4 = 0.25 * k, ik = 1.0 / k;
    const double *vp = vfree + p * 9, *vq = vfree + q * 9;
    auto moment = [&](int a, int b, double &jr, double &ji) {
        const double *va = vp + 3 * a, *vb = vq + 3 * b;
        const double vv = va[0] * vb[0] + va[1] * vb[1] + va[2] * vb[2];
        jr = S.sxyr + vv * S.s0r;
        ji = S.sxyi + vv * S.s0i;
        for (int c = 0; c < 3; ++c) {
            jr -= va[c] * S.syr[c] + vb[c] * S.sxr[c];
            ji -= va[c] * S.syi[c] + vb[c] * S.sxi[c];
        }
    };
    const int a = l / 3, b = l % 3;
    double Jr, Ji;
    moment(a, b, Jr, Ji);
    if (p == q && a != b) {
        // J_ab = J_ba for a self pair (swap the two integration variables);
        // take the mean so the stored block is symmetric to the last bit.
        double jr, ji;
        moment(b, a, jr, ji);
        Jr = 0.5 * (Jr + jr);
        Ji = 0.5 * (Ji + ji);
    }
    const double ss = double(sgn[p * 3 + a] * sgn[q * 3 + b]);
    const double lr = SPLIT ? ss * (-k4 * Ji) : ss * (-k4 * Ji + ik * S.s0i);
    const double li = SPLIT ? ss * (k4 * Jr) : ss * (k4 * Jr - ik * S.s0r);
    if (compact) {   // the pair's 3 x 3 block, pair after pair (near field of the fast operator)
        compact[at * 18 + l * 2 + 0] = lr;
        compact[at * 18 + l * 2 + 1] = li;
        return;
    }
    R *out = LB + 2 * bd.block(p, q, a, b);
    out[0] = R(lr);
    out[1] = R(li);
    if (SPLIT && l == 0) {
        R *vo = VS + 2 * bd.pair(p, q);
        vo[0] = R(ik * S.s0i);
        vo[1] = R(-ik * S.s0r);
    }
}

// ---------------------------------------------------------------------------
// 3. Assembly into the RWG matrix.
//
// Slot a of triangle p as it enters a local block: the row's first entry less
// that of column 0, and its place among the columns of another row, so that L of
// (row slot r, column slot c) is entry r.row + c.col of the scratch.
struct Slot {
    int64_t row;
    int32_t col;
};
__device__ __forceinline__ Slot slot_of(const Bands &bd, int32_t p, int32_t a)
{
    const int64_t I = p / TT;
    return { 9 * bd.base(I) + ((p % TT) * 3 + a) * 3 * bd.cols(I) - 3 * TT * I, 3 * p + a };
}

// T_mn from the four triangle pairs of (m, n); each is stored once, with the
// lower triangle as the row.  One block per stored tile (I, J), I <= J, of the
// packed symmetric matrix (or RPB of its TB / 4 groups of four rows); a wave takes
// every fourth row m of it and its lanes the 64 columns n, so that the row's slots are the same for the wave (scalar) and the
// column's are worked out once.  Bound by the gathers: four 16-byte reads an
// entry, each scratch entry used once but in lines that hold other tiles' too (7680
// unknowns: 4.7 GB fetched of 1.9 GB, 1.46 -> 0.77 ms).
template <typename R, int RPB>
__global__ __launch_bounds__(256) void k_assemble(int64_t N, Bands bd, int64_t nTz, const int4 *__restrict__ rwg4,
                                                  const R *__restrict__ LB, double2 *__restrict__ Z64,
                                                  float2 *__restrict__ Z32)
{
    typedef R V2 __attribute__((ext_vector_type(2)));
    int64_t I, J;
    tile_decode(blockIdx.x, nTz, I, J);
    const int64_t base = int64_t(blockIdx.x) * TB * TB;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t n = J * TB + lane;
    Slot np{ 0, 0 }, nm{ 0, 0 };
    if (n < N) {
        const int4 e = rwg4[n];
        np = slot_of(bd, e.x, e.z);
        nm = slot_of(bd, e.y, e.w);
    }
    const V2 *L = reinterpret_cast<const V2 *>(LB);
    auto read = [&](const Slot &r, const Slot &c) {
        return L[r.col <= c.col ? r.row + c.col : c.row + r.col];
    };
#pragma unroll 4
    for (int i = blockIdx.y * RPB; i < int(blockIdx.y + 1) * RPB; ++i) {
        const int64_t m = I * TB + wave + 4 * i;
        V2 z = { 0, 0 };
        if (m < N && n < N) {
            const int4 e = rwg4[m];
            const Slot mp = slot_of(bd, e.x, e.z), mm = slot_of(bd, e.y, e.w);
            const V2 pp = read(mp, np), mn = read(mm, nm), pm = read(mp, nm), mq = read(mm, np);
            z = (pp + mn) + (pm + mq);
        }
        const int64_t o = base + int64_t(wave + 4 * i) * TB + lane;
        if (Z64) Z64[o] = make_double2(double(z.x), double(z.y));
        if (Z32) Z32[o] = make_float2(float(z.x), float(z.y));
    }
}

// V' into packed F x F tiles (TB x TB, I <= J) from the per-pair values (p <= q;
// the other half by symmetry).
template <typename R>
__global__ __launch_bounds__(256) void k_assemble_v(int64_t F, Bands bd, int64_t nTv, const R *__restrict__ VS,
                                                    double2 *__restrict__ V64, float2 *__restrict__ V32)
{
    int64_t I, J;
    tile_decode(blockIdx.x, nTv, I, J);
    const int64_t base = int64_t(blockIdx.x) * TB * TB;
#pragma unroll 4
    for (int q = 0; q < TB * TB / 256; ++q) {
        const int e = threadIdx.x + 256 * q;
        int64_t a = I * TB + e / TB, b = J * TB + e % TB;
        R vr = 0, vi = 0;
        if (a < F && b < F) {
            if (a > b) { const int64_t t = a; a = b; b = t; }
            const R *src = VS + 2 * bd.pair(a, b);
            vr = src[0];
            vi = src[1];
        }
        if (V64) V64[base + e] = make_double2(double(vr), double(vi));
        if (V32) V32[base + e] = make_float2(float(vr), float(vi));
    }
}

// ---------------------------------------------------------------------------
// Plane-wave excitation:  e_m = sum_{p in m} (s_p/2) sum_i w_i (x_i - v_p).pol exp(-jk d.x_i)
// A lane keeps the 7 points of one side of its function for RB waves, whose
// directions and polarisations are the same for all lanes (scalar).  Bound by the
// sines and cosines (7680 unknowns, 256 waves: 79 us; a lane to each function and
// wave, points read again for each, 156).
template <int RB>
__global__ __launch_bounds__(256) void k_rhs(int64_t N, int64_t R, const int4 *__restrict__ rwg4,
                                             const int8_t *__restrict__ sgn, const double *__restrict__ cent,
                                             const double *__restrict__ loc, const double *__restrict__ vfree,
                                             const double *__restrict__ dirs, const double *__restrict__ pols,
                                             double k, double2 *__restrict__ B)
{
    const int64_t m = int64_t(blockIdx.x) * blockDim.x + threadIdx.x, r0 = int64_t(blockIdx.y) * RB;
    if (m >= N) return;
    const int4 e = rwg4[m];
    double br[RB], bi[RB];
#pragma unroll
    for (int u = 0; u < RB; ++u) br[u] = bi[u] = 0.0;
#pragma unroll 1
    for (int side = 0; side < 2; ++side) {
        const int64_t t = side ? e.y : e.x;
        const int a = side ? e.w : e.z;
        const double s = 0.5 * double(sgn[t * 3 + a]);
        double x[NQ][3], c[3], v[3];
#pragma unroll
        for (int q = 0; q < 3; ++q) {
            c[q] = cent[t * 3 + q];
            v[q] = vfree[t * 9 + a * 3 + q];
#pragma unroll
            for (int i = 0; i < NQ; ++i) x[i][q] = loc[(t * NQ + i) * 3 + q];
        }
#pragma unroll
        for (int u = 0; u < RB; ++u) {
            if (r0 + u >= R) break;
            const double *d = dirs + 3 * (r0 + u), *pl = pols + 3 * (r0 + u);
            double tr = 0.0, ti = 0.0;
#pragma unroll
            for (int i = 0; i < NQ; ++i) {
                double dv = 0.0, ph = 0.0;
#pragma unroll
                for (int q = 0; q < 3; ++q) {
                    dv += (x[i][q] - v[q]) * pl[q];
                    ph += d[q] * (c[q] + x[i][q]);
                }
                double sn, cs;
                sincos(k * ph, &sn, &cs);
                tr += c_w[i] * dv * cs;
                ti -= c_w[i] * dv * sn;
            }
            br[u] += s * tr;
            bi[u] += s * ti;
        }
    }
#pragma unroll
    for (int u = 0; u < RB; ++u)
        if (r0 + u < R) B[(r0 + u) * N + m] = make_double2(br[u], bi[u]);
}

// Radiation vector F(o) = int j(y) exp(jk o.y) dS = sum_t sum_i w_i J_t(y_i) exp(jk o.y_i),
// J_t(y) = sum_a x_{m(t,a)} s_a (y - v_a)/2 = b y - a with b = sum_a x_a s_a / 2 and
// a = sum_a x_a s_a v_a / 2 (y, v relative to the centroid), so that
//     F(o) = sum_t b_t P1_t(o) - a_t P0_t(o),  P0 = sum_i w_i exp(jk o.y_i), P1 = sum_i w_i y_i exp(..):
// the exponentials depend on the direction alone and the vectors enter by a
// contraction over the triangles.
//
// F itself, or with RCS the bistatic RCS (k^2 / (4 pi)) |r x F|^2 of direction r = o
// (unit): the part of F transverse to r, squared.
template <bool RCS, typename O>
__device__ inline void far_write(const double (&f)[6], const double (&o)[3], double k, O *__restrict__ out, int64_t at)
{
    if constexpr (RCS) {
        double dr = 0.0, di = 0.0, t2 = 0.0;
        for (int c = 0; c < 3; ++c) {
            dr += o[c] * f[2 * c];
            di += o[c] * f[2 * c + 1];
        }
        for (int c = 0; c < 3; ++c) {
            const double tr = f[2 * c] - dr * o[c], ti = f[2 * c + 1] - di * o[c];
            t2 += tr * tr + ti * ti;
        }
        out[at] = k * k / (4.0 * M_PI) * t2;
    } else {
        for (int c = 0; c < 3; ++c) out[at * 3 + c] = make_double2(f[2 * c], f[2 * c + 1]);
    }
}

// Few directions or a small mesh: one block per (vector, direction), its threads over the
// triangles, the exponentials evaluated for every vector again.  One launch and no
// work arrays (see farfield for the line).
template <bool RCS, typename O>
__global__ __launch_bounds__(256) void k_far_direct(int64_t F, int64_t N, int64_t M,
                                                    const int32_t *__restrict__ slot_m,
                                                    const int8_t *__restrict__ sgn, const double *__restrict__ cent,
                                                    const double *__restrict__ loc, const double *__restrict__ vfree,
                                                    const double *__restrict__ obs, double k,
                                                    const double2 *__restrict__ X, O *__restrict__ out)
{
    const int64_t mo = blockIdx.x, r = blockIdx.y;
    const double o[3] = { obs[3 * mo], obs[3 * mo + 1], obs[3 * mo + 2] };
    const double2 *x = X + r * N;
    double acc[6] = { 0, 0, 0, 0, 0, 0 };
    for (int64_t t = threadIdx.x; t < F; t += blockDim.x) {
        double br = 0.0, bi = 0.0, ar[3] = { 0, 0, 0 }, ai[3] = { 0, 0, 0 };   // J(y) = b y - a
        for (int a = 0; a < 3; ++a) {
            const double2 xa = x[slot_m[t * 3 + a]];
            const double sa = 0.5 * double(sgn[t * 3 + a]);
            br += sa * xa.x;
            bi += sa * xa.y;
            for (int c = 0; c < 3; ++c) {
                const double v = sa * vfree[t * 9 + a * 3 + c];
                ar[c] += v * xa.x;
                ai[c] += v * xa.y;
            }
        }
        for (int i = 0; i < NQ; ++i) {
            double y[3], ph = 0.0;
            for (int c = 0; c < 3; ++c) {
                y[c] = loc[(t * NQ + i) * 3 + c];
                ph += o[c] * (cent[t * 3 + c] + y[c]);
            }
            double sn, cs;
            sincos_reduced(k * ph, sn, cs);
            sn *= c_w[i];
            cs *= c_w[i];
            for (int c = 0; c < 3; ++c) {
                const double jr = br * y[c] - ar[c], ji = bi * y[c] - ai[c];
                acc[2 * c] += jr * cs - ji * sn;
                acc[2 * c + 1] += jr * sn + ji * cs;
            }
        }
    }
    __shared__ double red[6][4];
    for (int c = 0; c < 6; ++c) {
        for (int h = 32; h > 0; h >>= 1) acc[c] += __shfl_xor(acc[c], h, 64);
        if ((threadIdx.x & 63) == 0) red[c][threadIdx.x >> 6] = acc[c];
    }
    __syncthreads();
    if (threadIdx.x) return;
    double f[6];
    for (int c = 0; c < 6; ++c) f[c] = (red[c][0] + red[c][1]) + (red[c][2] + red[c][3]);
    far_write<RCS>(f, o, k, out, r * M + mo);
}

// (b, a) of every triangle and vector: 8 doubles at ((t R) + r) 8.
__global__ __launch_bounds__(256) void k_far_coef(int64_t F, int64_t N, int64_t R, const int32_t *__restrict__ slot_m,
                                                  const int8_t *__restrict__ sgn, const double *__restrict__ vfree,
                                                  const double2 *__restrict__ X, double *__restrict__ coef)
{
    const int64_t t = int64_t(blockIdx.x) * 256 + threadIdx.x, r = blockIdx.y;
    if (t >= F) return;
    double q[8] = { 0, 0, 0, 0, 0, 0, 0, 0 };
    for (int a = 0; a < 3; ++a) {
        const double2 x = X[r * N + slot_m[t * 3 + a]];
        const double s = 0.5 * double(sgn[t * 3 + a]);
        q[0] += s * x.x;
        q[1] += s * x.y;
        for (int c = 0; c < 3; ++c) {
            const double v = s * vfree[t * 9 + a * 3 + c];
            q[2 + 2 * c] += v * x.x;
            q[3 + 2 * c] += v * x.y;
        }
    }
    for (int i = 0; i < 8; ++i) coef[(t * R + r) * 8 + i] = q[i];
}

// Partial sums of F over the triangles of split z.  Lanes are 64 directions.  Of every
// FT = 8 triangles each of the four waves evaluates P0 and P1 of two into LDS, then
// takes its VW of the block's 4 VW vectors through all eight, with the coefficients in
// scalar registers: the exponentials are evaluated once for 32 vectors and no wave
// holds more than 8 vectors' sums.  FP64 vector issue bounds it: 7 sines and cosines
// per triangle and direction and 24 multiply-adds per vector (one block per vector and
// direction evaluated the exponentials for every vector; 7680 unknowns, 32 vectors,
// 361 directions: 3812 us, now 131; waves that kept their exponentials and 16 vectors each, one
// to a SIMD: 427 us).
constexpr int FT = 8;
template <int VW>
__global__ __launch_bounds__(256) void k_far_sum(int64_t F, int64_t R, int64_t M, int64_t per, const double *__restrict__ cent,
                                                 const double *__restrict__ loc, const double *__restrict__ obs, double k,
                                                 const double *__restrict__ coef, double *__restrict__ part)
{
    __shared__ double P[2][FT][8][64];
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t mo = int64_t(blockIdx.x) * 64 + lane, r0 = (int64_t(blockIdx.y) * 4 + w) * VW, ml = mo < M ? mo : M - 1;
    const double o[3] = { k * obs[3 * ml], k * obs[3 * ml + 1], k * obs[3 * ml + 2] };
    double f[VW][6];
#pragma unroll
    for (int r = 0; r < VW; ++r)
#pragma unroll
        for (int c = 0; c < 6; ++c) f[r][c] = 0.0;
    const int64_t t0 = int64_t(blockIdx.z) * per, t1 = min(F, t0 + per);
    int buf = 0;
    for (int64_t tb = t0; tb < t1; tb += FT, buf ^= 1) {
        const int nt = int(min(int64_t(FT), t1 - tb));
        for (int u = w; u < nt; u += 4) {
            const int64_t t = tb + u;
            const double *y = loc + t * NQ * 3;
            const double ph = o[0] * cent[3 * t] + o[1] * cent[3 * t + 1] + o[2] * cent[3 * t + 2];
            double p[8] = { 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0 };
#pragma unroll
            for (int i = 0; i < NQ; ++i) {
                double sn, cs;
                sincos_reduced(ph + (o[0] * y[3 * i] + o[1] * y[3 * i + 1] + o[2] * y[3 * i + 2]), sn, cs);
                sn *= c_w[i];
                cs *= c_w[i];
                p[0] += cs;
                p[1] += sn;
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    p[2 + 2 * c] += cs * y[3 * i + c];
                    p[3 + 2 * c] += sn * y[3 * i + c];
                }
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) P[buf][u][i][lane] = p[i];
        }
        __syncthreads();   // one for each buffer: the next pass writes the other
        for (int u = 0; u < nt; ++u) {
            double p[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) p[i] = P[buf][u][i][lane];
#pragma unroll
            for (int r = 0; r < VW; ++r) {
                const double *q = coef + ((tb + u) * R + min(r0 + r, R - 1)) * 8;   // beyond R: the last, not stored
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    f[r][2 * c] = __builtin_fma(q[0], p[2 + 2 * c], f[r][2 * c]);
                    f[r][2 * c] = __builtin_fma(-q[1], p[3 + 2 * c], f[r][2 * c]);
                    f[r][2 * c] = __builtin_fma(-q[2 + 2 * c], p[0], f[r][2 * c]);
                    f[r][2 * c] = __builtin_fma(q[3 + 2 * c], p[1], f[r][2 * c]);
                    f[r][2 * c + 1] = __builtin_fma(q[0], p[3 + 2 * c], f[r][2 * c + 1]);
                    f[r][2 * c + 1] = __builtin_fma(q[1], p[2 + 2 * c], f[r][2 * c + 1]);
                    f[r][2 * c + 1] = __builtin_fma(-q[2 + 2 * c], p[1], f[r][2 * c + 1]);
                    f[r][2 * c + 1] = __builtin_fma(-q[3 + 2 * c], p[0], f[r][2 * c + 1]);
                }
            }
        }
    }
    if (mo >= M) return;
#pragma unroll
    for (int r = 0; r < VW; ++r)
        if (r0 + r < R)
#pragma unroll
            for (int c = 0; c < 6; ++c) part[((int64_t(blockIdx.z) * R + r0 + r) * 6 + c) * M + mo] = f[r][c];
}

// The splits' sums in order, and what is asked for.
template <bool RCS, typename O>
__global__ __launch_bounds__(256) void k_far_out(int64_t nm, int64_t ld, int64_t splits, const double *__restrict__ part,
                                                const double *__restrict__ obs, double k, O *__restrict__ out)
{
    __shared__ double red[3][6][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;   // each wave a quarter of the splits
    const int64_t mo = int64_t(blockIdx.x) * 64 + lane, r = blockIdx.y, R = gridDim.y, q = (splits + 3) / 4;
    double f[6] = { 0, 0, 0, 0, 0, 0 };
    const double *p = part + r * 6 * nm + min(mo, nm - 1);
    const int64_t z1 = min(splits, (w + 1) * q);
    for (int64_t z = w * q; z < z1; z += 4) {   // four splits' loads at a time, beyond the last from the last
        double v[4][6];
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int c = 0; c < 6; ++c) v[u][c] = p[(min(z + u, z1 - 1) * R * 6 + c) * nm];
#pragma unroll
        for (int u = 0; u < 4; ++u)
#pragma unroll
            for (int c = 0; c < 6; ++c) f[c] += z + u < z1 ? v[u][c] : 0.0;
    }
    if (w)
        for (int c = 0; c < 6; ++c) red[w - 1][c][lane] = f[c];
    __syncthreads();
    if (w || mo >= nm) return;
    for (int u = 0; u < 3; ++u)
        for (int c = 0; c < 6; ++c) f[c] += red[u][c][lane];
    const double o[3] = { obs[3 * mo], obs[3 * mo + 1], obs[3 * mo + 2] };
    far_write<RCS>(f, o, k, out, r * ld + mo);
}

}  // namespace

// Weights of the triangle rule (relative to the area), for other kernels that
// integrate over the same quadrature points.
// The local 3 x 3 blocks L(p, a, q, b) of the flagged pairs (p <= q) of the
// mesh's list, pair after pair (18 doubles each: re, im of (a, b) row-major),
// with the fill's singular treatment.
void singular_blocks(const bie_op *op, const int32_t *pairs, int64_t npairs, double *out, hipStream_t s)
{
    if (npairs == 0) return;
    const TriDev &D = op->tri;
    hipLaunchKernelGGL((k_pairs_singular<double, false>), dim3(unsigned((npairs + 15) / 16)), dim3(256), 0, s, npairs,
                       Bands{ 0 }, pairs, D.cent, D.loc, D.vfree, D.verts, D.area, D.sgn, op->k, (double *)nullptr,
                       (double *)nullptr, out);
    BIE_HIP(hipGetLastError());
}

void quad_weights(double *w)
{
    const Rule rule = make_rule();
    for (int i = 0; i < NQ; ++i) w[i] = rule.w[i];
}

// Per-triangle tables on the device, in the given order or that of the triangles'
// lowest RWG function: consecutive functions then lie on nearly consecutive triangles, and
// the assembly finds most local blocks of a row (p <= q) in one run.  Quadrature
// points and free vertices relative to the triangle centroid (keeps FP32 local
// arithmetic accurate).
void upload_triangles(bie_op *op, hipStream_t s, const std::vector<int32_t> *given)
{
    const Mesh &M = op->mesh;
    const int64_t F = M.F;
    const Rule rule = make_rule();
    TriDev &D = op->tri;
    D.rank.assign(F, -1);
    std::vector<int32_t> order;
    order.reserve(F);
    if (given) {
        order = *given;
        for (int64_t r = 0; r < F; ++r) D.rank[order[r]] = int32_t(r);
    }
    for (int64_t m = 0; m < M.N && !given; ++m)
        for (int side = 0; side < 2; ++side) {
            const int32_t t = M.edges[4 * m + 2 + side];
            if (D.rank[t] >= 0) continue;
            D.rank[t] = int32_t(order.size());
            order.push_back(t);
        }
    // one host image of the tables, copied at once
    size_t bytes = 0;
    auto place = [&](size_t n, size_t size) {
        const size_t at = bytes;
        bytes += (n * size + 255) / 256 * 256;
        return at;
    };
    const size_t d = sizeof(double), i4 = sizeof(int32_t);
    const size_t o_cent = place(3 * F, d), o_loc = place(3 * NQ * F, d), o_vf = place(9 * F, d), o_vt = place(9 * F, d),
                 o_area = place(F, d), o_rad = place(F, d), o_sgn = place(3 * F, 1), o_slot = place(3 * F, i4),
                 o_edges = place(4 * M.N, i4);
    std::vector<char> image(bytes);
    auto doubles = [&](size_t o) { return reinterpret_cast<double *>(image.data() + o); };
    auto ints = [&](size_t o) { return reinterpret_cast<int32_t *>(image.data() + o); };
    double *cent = doubles(o_cent), *loc = doubles(o_loc), *vf = doubles(o_vf), *vt = doubles(o_vt),
           *area = doubles(o_area), *rad = doubles(o_rad);
    int8_t *sgn = reinterpret_cast<int8_t *>(image.data() + o_sgn);
    int32_t *slot = ints(o_slot), *r4 = ints(o_edges);   // r4: (c+, c-, slot of m in c+, slot of m in c-)
    for (int64_t r = 0; r < F; ++r) {
        const int64_t t = order[r];
        const double *v[3] = { &M.V[3 * M.T[3 * t]], &M.V[3 * M.T[3 * t + 1]], &M.V[3 * M.T[3 * t + 2]] };
        const double *c = &M.cent[3 * t];
        area[r] = M.area[t];
        rad[r] = 0.0;
        for (int i = 0; i < NQ; ++i) {
            double d2 = 0.0;
            for (int d = 0; d < 3; ++d) {
                const double x = rule.bary[i][0] * v[0][d] + rule.bary[i][1] * v[1][d] + rule.bary[i][2] * v[2][d];
                loc[(r * NQ + i) * 3 + d] = x - c[d];
                d2 += (x - c[d]) * (x - c[d]);
            }
            rad[r] = std::max(rad[r], std::sqrt(d2));
        }
        D.max_rad = std::max(D.max_rad, rad[r]);
        for (int a = 0; a < 3; ++a) {
            sgn[r * 3 + a] = M.slot_s[3 * t + a];
            slot[r * 3 + a] = M.slot_m[3 * t + a];
            cent[r * 3 + a] = c[a];
            for (int d = 0; d < 3; ++d) {
                vf[r * 9 + a * 3 + d] = v[a][d] - c[d];
                vt[r * 9 + a * 3 + d] = v[a][d];
            }
        }
    }
    for (int64_t m = 0; m < M.N; ++m) {
        const int32_t tp = M.edges[4 * m + 2], tm = M.edges[4 * m + 3];
        int sp = -1, sm = -1;
        for (int a = 0; a < 3; ++a) {
            if (M.slot_m[3 * tp + a] == m) sp = a;
            if (M.slot_m[3 * tm + a] == m) sm = a;
        }
        r4[4 * m + 0] = D.rank[tp]; r4[4 * m + 1] = D.rank[tm]; r4[4 * m + 2] = sp; r4[4 * m + 3] = sm;
    }
    BIE_HIP(device_malloc(&D.mem, bytes));
    BIE_HIP(hipMemcpy(D.mem, image.data(), bytes, hipMemcpyHostToDevice));
    auto dev = [&](auto *&p, size_t o) { p = reinterpret_cast<std::remove_reference_t<decltype(p)>>(static_cast<char *>(D.mem) + o); };
    dev(D.cent, o_cent);
    dev(D.loc, o_loc);
    dev(D.vfree, o_vf);
    dev(D.verts, o_vt);
    dev(D.area, o_area);
    dev(D.rad, o_rad);
    dev(D.sgn, o_sgn);
    dev(D.slot_m, o_slot);
    dev(D.edges, o_edges);
    (void)s;
}

template <typename R, bool SPLIT>
static void fill_launch(bie_op *op, const Bands &bd, const int32_t *pairs, int64_t npairs, void *LB,
                        void *VS, bool want64, bool want32, hipStream_t s)
{
    const Mesh &M = op->mesh;
    const TriDev &D = op->tri;
    // measurement records: 6 regular pairs (columns = triangle pairs p <= q), 7
    // flagged pairs, 8 assembly (columns = unknowns)
    const int rec_reg = sizeof(R) == 8 ? 6 : 9;
    prof_begin(rec_reg, s, M.F * (M.F + 1) / 2);
    // enough blocks for four waves on every SIMD: small meshes split the rows of
    // a band (16 rows per block at 320 triangles left 20 blocks: 100 us, 29 us split)
    const int64_t blocks = bd.total() / (TT * 256) + bd.Fp / TT;
    const unsigned nz = unsigned(std::min<int64_t>(TT, std::max<int64_t>(1, 1024 / blocks)));
    const dim3 grid(unsigned((bd.Fp + 255) / 256), unsigned(bd.Fp / TT), nz);
    if constexpr (sizeof(R) == 8)
        hipLaunchKernelGGL((k_pairs_regular<R, SPLIT, true>), grid, dim3(256), 0, s, M.F, bd, D.cent, D.loc, D.vfree,
                           D.sgn, D.rad, op->k, (R *)LB, (R *)VS);
    if (sizeof(R) == 4 || op->k * 2.0 * D.max_rad > NARROW_PHASE)
        hipLaunchKernelGGL((k_pairs_regular<R, SPLIT, false>), grid, dim3(256), 0, s, M.F, bd, D.cent, D.loc, D.vfree,
                           D.sgn, D.rad, op->k, (R *)LB, (R *)VS);
    prof_end(rec_reg, s);
    prof_begin(7, s, npairs);
    if (npairs)
        hipLaunchKernelGGL((k_pairs_singular<R, SPLIT>), dim3(unsigned((npairs + 15) / 16)), dim3(256), 0, s, npairs,
                           bd, pairs, D.cent, D.loc, D.vfree, D.verts, D.area, D.sgn, op->k, (R *)LB, (R *)VS);
    prof_end(7, s);
    prof_begin(8, s, M.N);
    // few tiles: four blocks each, so that every CU has some (480 unknowns, 36 tiles: 21 -> 8 us)
    if (op->pk.ntiles < 1024)
        hipLaunchKernelGGL((k_assemble<R, TB / 16>), dim3(unsigned(op->pk.ntiles), 4), dim3(256), 0, s, M.N, bd, op->pk.nT,
                           (const int4 *)D.edges, (const R *)LB, want64 ? (double2 *)op->Z64 : nullptr,
                           want32 ? (float2 *)op->Z32 : nullptr);
    else
        hipLaunchKernelGGL((k_assemble<R, TB / 4>), dim3(unsigned(op->pk.ntiles)), dim3(256), 0, s, M.N, bd, op->pk.nT,
                           (const int4 *)D.edges, (const R *)LB, want64 ? (double2 *)op->Z64 : nullptr,
                           want32 ? (float2 *)op->Z32 : nullptr);
    prof_end(8, s);
    if (SPLIT)
        hipLaunchKernelGGL(k_assemble_v<R>, dim3(unsigned(op->pkv.ntiles)), dim3(256), 0, s, M.F, bd, op->pkv.nT,
                           (const R *)VS, want64 ? (double2 *)op->V64 : nullptr, want32 ? (float2 *)op->V32 : nullptr);
}

// The matrix (or, for a star-split operator, T_A' and V') into the packed
// arrays the operator holds.
void fill_matrix(bie_op *op, bool fp64_regular, bool want64, bool want32, hipStream_t s)
{
    const Mesh &M = op->mesh;
    const int64_t F = M.F;
    const Bands bd{ (F + TT - 1) / TT * TT };
    const size_t elem = fp64_regular ? sizeof(double) : sizeof(float);
    PoolBlock lb(s), vs(s);
    const int32_t *pairs = op->flagged;
    const int64_t npairs = int64_t(M.near.size() / 2);
    lb.get(size_t(bd.total()) * 9 * 2 * elem);
    if (op->star) vs.get(size_t(bd.total()) * 2 * elem);
    if (fp64_regular) {
        if (op->star) fill_launch<double, true>(op, bd, pairs, npairs, lb.p, vs.p, want64, want32, s);
        else fill_launch<double, false>(op, bd, pairs, npairs, lb.p, vs.p, want64, want32, s);
    } else {
        if (op->star) fill_launch<float, true>(op, bd, pairs, npairs, lb.p, vs.p, want64, want32, s);
        else fill_launch<float, false>(op, bd, pairs, npairs, lb.p, vs.p, want64, want32, s);
    }
    BIE_HIP(hipGetLastError());
    BIE_HIP(hipStreamSynchronize(s));
    (void)hipFree(op->flagged);   // not read again
    op->flagged = nullptr;
}

void rhs_planewave(const bie_op *op, const double *dirs, const double *pols, int64_t R, void *B, hipStream_t s)
{
    const int64_t N = op->mesh.N;
    double *dd = nullptr;
    BIE_HIP(device_malloc(&dd, 6 * R * sizeof(double)));
    BIE_HIP(hipMemcpy(dd, dirs, 3 * R * sizeof(double), hipMemcpyHostToDevice));
    BIE_HIP(hipMemcpy(dd + 3 * R, pols, 3 * R * sizeof(double), hipMemcpyHostToDevice));
    const TriDev &D = op->tri;
    // four waves per lane once that leaves four blocks for each CU, else one for more blocks
    const unsigned nb = unsigned((N + 255) / 256);
    auto rhs = [&](auto kern, int rb) {
        hipLaunchKernelGGL(kern, dim3(nb, unsigned((R + rb - 1) / rb)), dim3(256), 0, s, N, R, (const int4 *)D.edges,
                           D.sgn, D.cent, D.loc, D.vfree, dd, dd + 3 * R, op->k, (double2 *)B);
    };
    if (nb * R >= 4096) rhs(k_rhs<4>, 4);
    else rhs(k_rhs<1>, 1);
    BIE_HIP(hipGetLastError());
    BIE_HIP(hipStreamSynchronize(s));
    hipFree(dd);
}

void farfield(const bie_op *op, const void *X, int64_t R, const double *obs, int64_t M, void *out, bool rcs,
              hipStream_t s)
{
    const TriDev &D = op->tri;
    const int64_t F = op->mesh.F, N = op->mesh.N;
    // Vectors per wave: as many as the registers hold, the fewest that cover R.
    // Triangle splits: two blocks on each of the 256 CUs.  The coefficients and the
    // partial sums of one pass fill at most 64 MB each; more vectors or directions
    // go in several passes over the same buffers, and where even that is not to be
    // had in much smaller ones.
    struct Plan {
        int VW;
        int64_t nr, nm, per, splits;
        size_t coef, part;
    };
    auto plan = [&](int64_t limit) {
        Plan p;
        p.nr = std::min(R, std::max<int64_t>(1, limit / (8 * F)));
        p.VW = p.nr > 16 ? 8 : p.nr > 8 ? 4 : p.nr > 4 ? 2 : 1;
        const int64_t by = (p.nr + 4 * p.VW - 1) / (4 * p.VW), most = std::max<int64_t>(64, limit / (6 * p.nr) / 64 * 64);
        p.nm = std::min(M, most);
        const int64_t bx = (p.nm + 63) / 64;
        const int64_t want = std::max<int64_t>(1, std::min({ (F + 15) / 16, 512 / (bx * by), most / p.nm }));
        p.per = (F + want - 1) / want;
        p.splits = (F + p.per - 1) / p.per;
        p.coef = size_t(8 * F * p.nr);
        p.part = size_t(6 * p.splits * p.nr * p.nm);
        return p;
    };
    double *w = nullptr;
    Plan p = {};
    const size_t nobs = size_t(3 * M);
    // One block per (vector, direction) where that is estimated faster (us: its chain over the
    // triangles or all blocks' issue, against two more launches, their chain and the
    // coefficients; wall time direct / three launches: 72 unknowns, one vector and direction 35 /
    // 48; 480, 512 vectors, one direction 41 / 98, 64 directions 371 / 102; 7200, 512 vectors, 4
    // directions 393 / 831, 16 1440 / 816; 30720, one vector, 361 directions 349 / 292).
    const double fr = double(F) * double(R);
    if (std::max(0.01 * double(F), 3.3e-5 * fr * double(M)) < 16.0 + 0.002 * double(F) + 2e-4 * fr) {
        BIE_HIP(device_malloc(&w, nobs * sizeof(double)));
        hipError_t e = hipMemcpy(w, obs, nobs * sizeof(double), hipMemcpyHostToDevice);
        auto go = [&](auto kern, auto *to) {
            hipLaunchKernelGGL(kern, dim3(unsigned(M), unsigned(R)), dim3(256), 0, s, F, N, M, D.slot_m, D.sgn, D.cent,
                               D.loc, D.vfree, w, op->k, (const double2 *)X, to);
        };
        if (e == hipSuccess) {
            if (rcs) go(k_far_direct<true, double>, static_cast<double *>(out));
            else go(k_far_direct<false, double2>, static_cast<double2 *>(out));
            e = hipGetLastError();
        }
        const hipError_t e2 = hipStreamSynchronize(s);
        (void)hipFree(w);
        BIE_HIP(e);
        BIE_HIP(e2);
        return;
    }
    hipError_t e = hipErrorOutOfMemory;
    for (int64_t limit : { int64_t(1) << 23, int64_t(1) << 19, int64_t(0) }) {
        p = plan(limit);
        e = device_malloc(&w, (nobs + p.coef + p.part) * sizeof(double));
        if (e != hipErrorOutOfMemory) break;
        (void)hipGetLastError();
    }
    BIE_HIP(e);
    double *dobs = w, *coef = w + nobs, *part = coef + p.coef;
    e = hipMemcpy(dobs, obs, nobs * sizeof(double), hipMemcpyHostToDevice);
    for (int64_t r0 = 0; r0 < R && e == hipSuccess; r0 += p.nr) {
        const int64_t nr = std::min(p.nr, R - r0);
        hipLaunchKernelGGL(k_far_coef, dim3(unsigned((F + 255) / 256), unsigned(nr)), dim3(256), 0, s, F, N, nr, D.slot_m,
                           D.sgn, D.vfree, (const double2 *)X + r0 * N, coef);
        for (int64_t m0 = 0; m0 < M; m0 += p.nm) {
            const int64_t nm = std::min(p.nm, M - m0);
            const unsigned bx = unsigned((nm + 63) / 64), by = unsigned((nr + 4 * p.VW - 1) / (4 * p.VW));
            auto sum = [&](auto kern) {
                hipLaunchKernelGGL(kern, dim3(bx, by, unsigned(p.splits)), dim3(256), 0, s, F, nr, nm, p.per, D.cent,
                                   D.loc, dobs + 3 * m0, op->k, coef, part);
            };
            if (p.VW == 8) sum(k_far_sum<8>);
            else if (p.VW == 4) sum(k_far_sum<4>);
            else if (p.VW == 2) sum(k_far_sum<2>);
            else sum(k_far_sum<1>);
            auto put = [&](auto kern, auto *to) {
                hipLaunchKernelGGL(kern, dim3(bx, unsigned(nr)), dim3(256), 0, s, nm, M, p.splits, part, dobs + 3 * m0,
                                   op->k, to);
            };
            if (rcs) put(k_far_out<true, double>, static_cast<double *>(out) + r0 * M + m0);
            else put(k_far_out<false, double2>, static_cast<double2 *>(out) + (r0 * M + m0) * 3);
        }
        e = hipGetLastError();
    }
    const hipError_t e2 = hipStreamSynchronize(s);
    (void)hipFree(w);
    BIE_HIP(e);
    BIE_HIP(e2);
}

}  // namespace bie
