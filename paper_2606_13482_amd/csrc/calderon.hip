// Multiplicative Calderon preconditioner of the EFIE (Andriulli et al., IEEE TAP
// 56(8), 2008), which the paper uses in all of its simulations (Sec. VI-A, remark
// on the star-split operator; Sec. VII, setup of the results) without restating it.
//
// M = -G^{-1} T_BC G^{-T}, stored like T in packed symmetric FP64 tiles (M is
// complex symmetric because T_BC is), so that one preconditioned product costs
// two packed products.  Pieces:
//   * barycentric refinement (host): each triangle cut into six by its centroid
//     and edge midpoints; vertices = original, then the midpoint of RWG edge m at
//     nv + m, then the centroid of triangle t at nv + N + t;
//   * BC functions (host): b_m is the combination of refined RWG functions on
//     the dual cells (refined triangles around a vertex) of the two ends of edge
//     m with charge +1/A(hi) spread uniformly over the cell of the higher vertex
//     and -1/A(lo) over the lower one's, flux 1/2 through each of the two refined
//     edges from the midpoint of m to the centroids of c+ and c-, and no flux
//     through the two halves of edge m.  Walking around a cell from the child
//     next to one half of the dual edge, the flux through each radial edge is
//     the previous one plus the child's share of the charge;
//   * mixed Gram matrix G_mn = <n x b_m, f_n> (host, CSR): exact with the
//     three-edge-midpoint rule on each refined triangle (quadratic integrand);
//   * T_BC = C Z_b C^T (device), Z_b the EFIE matrix of the refined mesh, from the
//     local blocks of the refined triangle pairs, cell by cell, without Z_b;
//   * G^{-1} applied to all N columns at once by Chebyshev iteration on the
//     interval that holds G's spectrum (CG on the normal equations if it fails),
//     twice with a transpose in between, on row-major blocks so that the sparse
//     products read whole rows of 64 columns.
#include <algorithm>
#include <cstdlib>
#include <cstring>
#include <chrono>
#include <map>
#include <memory>
#include <mutex>

#include "bie_internal.hpp"
#include "pairs.hpp"

struct bie_calderon {
    const bie_op *op = nullptr;   // operator it was built for (mesh and k)
    bie_op *view = nullptr;       // N x N packed FP64 tiles of M, products through the packed kernels
    bie_op *tm = nullptr;         // T M (dense, split-BF16 copy only) for the preconditioned block products
    void *tmp = nullptr;          // 2 x tmp_R x N complex128 for the preconditioned solve
    int64_t tmp_R = 0;
    bie_calderon_info info{};
};

namespace bie {
namespace {

constexpr int CT = 256;

std::mutex g_setup_mu;   // one setup at a time: a setup's work arrays are the largest part of its memory

struct Csr {
    std::vector<int64_t> ptr;
    std::vector<int32_t> idx;
    std::vector<double> val;
};

struct CsrDev {
    int64_t rows = 0;
    int64_t *ptr = nullptr;
    int32_t *idx = nullptr;
    double *val = nullptr;
    void upload(const Csr &c)
    {
        rows = int64_t(c.ptr.size()) - 1;
        BIE_HIP(device_malloc(&ptr, c.ptr.size() * sizeof(int64_t)));
        BIE_HIP(device_malloc(&idx, std::max<size_t>(1, c.idx.size()) * sizeof(int32_t)));
        BIE_HIP(device_malloc(&val, std::max<size_t>(1, c.val.size()) * sizeof(double)));
        BIE_HIP(hipMemcpy(ptr, c.ptr.data(), c.ptr.size() * sizeof(int64_t), hipMemcpyHostToDevice));
        BIE_HIP(hipMemcpy(idx, c.idx.data(), c.idx.size() * sizeof(int32_t), hipMemcpyHostToDevice));
        BIE_HIP(hipMemcpy(val, c.val.data(), c.val.size() * sizeof(double), hipMemcpyHostToDevice));
    }
    ~CsrDev()
    {
        if (ptr) (void)hipFree(ptr);
        if (idx) (void)hipFree(idx);
        if (val) (void)hipFree(val);
    }
};

// ----------------------------------------------------------------------------- kernels

// Y = A X for a real CSR matrix A and n x nc complex matrices stored row-major
// (entry (i, c) at i nc + c): a wave takes 64 consecutive columns of one row, so
// each nonzero reads 1 KiB contiguously.  Grid: rows x column blocks, rows
// fastest, so that the workgroups in flight share one column slice of X (kept in
// the last-level cache while they walk the rows).
__global__ __launch_bounds__(CT) void k_csr_rm(const int64_t *__restrict__ ptr, const int32_t *__restrict__ idx,
                                               const double *__restrict__ val, int64_t nc, const double2 *__restrict__ X,
                                               double2 *__restrict__ Y)
{
    const int64_t c = int64_t(blockIdx.y) * CT + threadIdx.x, i = blockIdx.x;
    if (c >= nc) return;
    double re = 0.0, im = 0.0;
    for (int64_t k = ptr[i]; k < ptr[i + 1]; ++k) {
        const double a = val[k];
        const double2 v = X[int64_t(idx[k]) * nc + c];
        re += a * v.x;
        im += a * v.y;
    }
    Y[i * nc + c] = make_double2(re, im);
}

__global__ void k_fill0(int64_t n, double2 *__restrict__ a)
{
    for (int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; e < n; e += int64_t(gridDim.x) * blockDim.x)
        a[e] = make_double2(0.0, 0.0);
}

// Row-major n x n: partial sums over the rows i = s, s + S, ... of |X(i, c)|^2
// (grid: column blocks x S slices), then their sum per column.
__global__ __launch_bounds__(CT) void k_colsq_part(int64_t n, const double2 *__restrict__ X, double *__restrict__ part)
{
    const int64_t c = int64_t(blockIdx.x) * CT + threadIdx.x;
    if (c >= n) return;
    double s = 0.0;
    for (int64_t i = blockIdx.y; i < n; i += gridDim.y) {
        const double2 v = X[i * n + c];
        s += v.x * v.x + v.y * v.y;
    }
    part[int64_t(blockIdx.y) * n + c] = s;
}

__global__ __launch_bounds__(CT) void k_colsq_fin(int64_t n, int S, const double *__restrict__ part,
                                                  double *__restrict__ out)
{
    const int64_t c = int64_t(blockIdx.x) * CT + threadIdx.x;
    if (c >= n) return;
    double s = 0.0;
    for (int k = 0; k < S; ++k) s += part[int64_t(k) * n + c];
    out[c] = s;
}

// CGNR step, per column c of row-major n x n blocks: alpha = zz / ww; X += alpha P;
// R -= alpha W (grid-stride over the entries).
__global__ __launch_bounds__(CT) void k_cg_xr(int64_t n, const double *__restrict__ zz, const double *__restrict__ ww,
                                              const double2 *__restrict__ P, const double2 *__restrict__ W,
                                              double2 *__restrict__ X, double2 *__restrict__ Rr)
{
    for (int64_t e = int64_t(blockIdx.x) * CT + threadIdx.x; e < n * n; e += int64_t(gridDim.x) * CT) {
        const int64_t c = e % n;
        const double a = ww[c] > 0.0 ? zz[c] / ww[c] : 0.0;
        const double2 p = P[e], w = W[e];
        double2 x = X[e], r = Rr[e];
        x.x += a * p.x;
        x.y += a * p.y;
        r.x -= a * w.x;
        r.y -= a * w.y;
        X[e] = x;
        Rr[e] = r;
    }
}

// CGNR direction, per column c of row-major blocks: beta = zn / zz; P = Z + beta P.
__global__ __launch_bounds__(CT) void k_cg_p(int64_t n, const double *__restrict__ zn, const double *__restrict__ zz,
                                             const double2 *__restrict__ Zv, double2 *__restrict__ P)
{
    for (int64_t e = int64_t(blockIdx.x) * CT + threadIdx.x; e < n * n; e += int64_t(gridDim.x) * CT) {
        const int64_t c = e % n;
        const double b = zz[c] > 0.0 ? zn[c] / zz[c] : 0.0;
        const double2 z = Zv[e], p = P[e];
        P[e] = make_double2(z.x + b * p.x, z.y + b * p.y);
    }
}

// B = A^T for column-major n x n complex matrices (32 x 32 tiles through LDS).
__global__ __launch_bounds__(256) void k_transpose(int64_t n, const double2 *__restrict__ A, double2 *__restrict__ B)
{
    __shared__ double2 t[32][33];
    const int64_t c0 = int64_t(blockIdx.y) * 32, r0 = int64_t(blockIdx.x) * 32;
    for (int k = threadIdx.y; k < 32; k += 8) {
        const int64_t r = r0 + threadIdx.x, c = c0 + k;
        if (r < n && c < n) t[k][threadIdx.x] = A[c * n + r];
    }
    __syncthreads();
    for (int k = threadIdx.y; k < 32; k += 8) {
        const int64_t r = c0 + threadIdx.x, c = r0 + k;   // B(r, c) = A(c, r)
        if (r < n && c < n) B[c * n + r] = t[threadIdx.x][k];
    }
}

// Packed symmetric tiles (I <= J, row-major tiles of TB x TB, row-major over the
// upper triangle) of s (A + A^T)/2 for a dense column-major n x n matrix A.
__global__ __launch_bounds__(256) void k_pack_sym(int64_t n, int64_t nT, const double2 *__restrict__ A, double s,
                                                  double2 *__restrict__ Zp)
{
    const int64_t I = blockIdx.y, J = blockIdx.x;
    if (J < I) return;
    double2 *tile = Zp + (I * nT - I * (I - 1) / 2 + (J - I)) * int64_t(TB * TB);
    for (int e = threadIdx.x; e < TB * TB; e += 256) {
        const int64_t i = I * TB + e / TB, j = J * TB + e % TB;
        double2 v = make_double2(0.0, 0.0);
        if (i < n && j < n) {
            const double2 a = A[j * n + i], b = A[i * n + j];
            v = make_double2(0.5 * s * (a.x + b.x), 0.5 * s * (a.y + b.y));
        }
        tile[e] = v;
    }
}

// Columns j0 .. j0 + nc - 1 of the n x n identity, dense (n entries per column).
__global__ __launch_bounds__(256) void k_unit_cols(int64_t n, int64_t j0, int64_t nc, double2 *__restrict__ X)
{
    for (int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; e < n * nc; e += int64_t(gridDim.x) * blockDim.x)
        X[e] = make_double2(e % n == j0 + e / n ? 1.0 : 0.0, 0.0);
}

__global__ __launch_bounds__(256) void k_add_cols(int64_t n, const double2 *__restrict__ a, double2 *__restrict__ x)
{
    for (int64_t e = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; e < n; e += int64_t(gridDim.x) * blockDim.x) {
        const double2 v = a[e];
        double2 y = x[e];
        y.x += v.x;
        y.y += v.y;
        x[e] = y;
    }
}

// ----------------------------------------------------------------------------- the dual matrix
//
// T_BC without the refined mesh's matrix.  The children of a vertex's dual cell (its
// refined triangles, one after another in the device order) carry the halves of the
// BC functions of the vertex's edges: with c_i(s, a) the coefficient, in the i-th of
// those functions, of the refined RWG function of slot a of child s,
//     D_vw(i, j) = sum_{s in v, a} sum_{t in w, b} c_i(s, a) L(s, a; t, b) c_j(t, b)
// and T_BC(m, n) is the sum of the four D over the end vertices of m and of n.  A
// block of the kernel takes one cell v and up to CB children t of whole cells w >= v,
// one per lane; a lane goes through the children s of v (their data in scalar
// registers; staged in LDS they cost a block per CU, 8.7 ms), adding c_i(s, .) L(s; t) to E_i(b) in registers, and the block then
// contracts E with c_j through LDS.  Each pair is computed once and leaves 36
// numbers per cell pair instead of nine per triangle pair: the refined matrix
// (36 N^2 entries), its pair scratch and its dense copy, 1440 N^2 bytes with a fill,
// an assembly, a copy and a gather over them, are 32 N^2 bytes and one kernel.
// FP64 vector issue bounds it: 2592
// unknowns, 53.7 M refined pairs 6.9 ms; those four took 20 ms.
constexpr int CB = 128;   // children t per block
// CI functions of v per block (a vertex with more edges takes more blocks): 6, the
// degree of a regular mesh's vertices, when none has more; otherwise 8.  E lies in
// LDS, 48 CI bytes a lane, which sets the waves in flight: 2 per SIMD with 6, 1.5
// with 8; in registers it left one (2592 unknowns: 7.9 ms with 8, 6.9 with 6 here).

// One cell, or a part of one with more than CB children: children t0 .. t0 + nt - 1,
// deg edges, their rows h0 .. h0 + deg - 1 among all cells' rows, coefficients
// c_i(s, a) at cf + ((s - t0) dp + i) 3 + a (dp: deg rounded up to CI,
// zeros beyond).
struct Cell {
    int32_t t0, nt, deg, dp;
    int64_t h0, cf;
};

// NARROW: the pairs within NARROW_PHASE and the flagged ones, D stored; otherwise
// the rest, added to it.
template <bool NARROW, int CI>
__global__ __launch_bounds__(CB) __attribute__((amdgpu_waves_per_eu(2))) void k_cells(const Cell *__restrict__ cells, const int32_t *__restrict__ group,
                                              const int32_t *__restrict__ cell_of, const int32_t *__restrict__ row_cell,
                                              const double *__restrict__ coef, const int64_t *__restrict__ rowoff,
                                              const double *__restrict__ cent, const double *__restrict__ loc,
                                              const double *__restrict__ vfree, const int8_t *__restrict__ sgn,
                                              const double *__restrict__ rad, const double *__restrict__ longest,
                                              const double *__restrict__ qw, const int64_t *__restrict__ fptr,
                                              const int32_t *__restrict__ fq, const double *__restrict__ fblk,
                                              double near_factor, double k, double2 *__restrict__ D)
{
    __shared__ double2 sE[CI * 3][CB];
    __shared__ double sw[QPTS], sw4[QPTS];
    const int32_t v = blockIdx.y, w0 = group[blockIdx.x], w1 = group[blockIdx.x + 1];   // cells w0 .. w1 - 1
    if (w1 <= v) return;
    const Cell V = cells[v];
    const int i0 = blockIdx.z * CI;
    if (i0 >= V.deg) return;
    const int tid = threadIdx.x;
    if (tid < QPTS) {
        sw[tid] = qw[tid];
        sw4[tid] = qw[tid] / (4.0 * M_PI);
    }
    __syncthreads();
    const int32_t tb = cells[w0].t0, te = cells[w1 - 1].t0 + cells[w1 - 1].nt;
    const int32_t t = tb + tid;
    const bool live = t < te && cell_of[t] >= v;
    for (int i = 0; i < CI * 3; ++i) sE[i][tid] = make_double2(0.0, 0.0);
    double y[QPTS][3], ct[3] = { 0.0, 0.0, 0.0 }, rt = 0.0, lt = 0.0;
    if (live) {
#pragma unroll
        for (int j = 0; j < QPTS; ++j)
#pragma unroll
            for (int c = 0; c < 3; ++c) y[j][c] = loc[(int64_t(t) * QPTS + j) * 3 + c];
        for (int c = 0; c < 3; ++c) ct[c] = cent[3 * int64_t(t) + c];
        rt = rad[t];
        lt = longest[t];
    }
    const auto yq = [&](int j, int c) { return y[j][c]; };
    const double k4 = 0.25 * k, ik = 1.0 / k;
    if (live) {
#pragma unroll 1
        for (int32_t s = V.t0; s < V.t0 + V.nt; ++s) {   // uniform: child s comes through scalar registers
            const double d[3] = { cent[3 * int64_t(s)] - ct[0], cent[3 * int64_t(s) + 1] - ct[1],
                                  cent[3 * int64_t(s) + 2] - ct[2] };
            const double dd = d[0] * d[0] + d[1] * d[1] + d[2] * d[2], thr = near_factor * fmax(longest[s], lt);
            // a flagged pair shares a vertex (centroids within 4/3 of the longest edge) or is near
            const double *blk = nullptr;
            if (dd < thr * thr * (1.0 + 1e-9)) {
                const int32_t p = min(s, t), q = max(s, t);
                int64_t lo = fptr[p], hi = fptr[p + 1];
                const int64_t end = hi;
                while (lo < hi) {
                    const int64_t mid = (lo + hi) >> 1;
                    if (fq[mid] < q) lo = mid + 1;
                    else hi = mid;
                }
                if (lo < end && fq[lo] == q) blk = fblk + lo * 18;
            }
            const bool narrow = k * (rad[s] + rt) <= NARROW_PHASE;
            const bool mine = NARROW ? narrow || blk : !narrow && !blk;
            if (!__any(mine)) continue;
            PairSums<double> S;
            pair_sums<double, NARROW>(loc + int64_t(s) * QPTS * 3, yq, d, k, sw, sw4, S);
            double vb[3][3], sb[3];
#pragma unroll
            for (int b = 0; b < 3; ++b) {
                sb[b] = double(sgn[3 * int64_t(t) + b]);
#pragma unroll
                for (int c = 0; c < 3; ++c) vb[b][c] = vfree[9 * int64_t(t) + 3 * b + c];
            }
            const double *cf = coef + V.cf + (int64_t(s - V.t0) * V.dp + i0) * 3;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                const double va[3] = { vfree[9 * int64_t(s) + 3 * a], vfree[9 * int64_t(s) + 3 * a + 1],
                                       vfree[9 * int64_t(s) + 3 * a + 2] };
                double lr[3], li[3];
                local_row<double, false>(S, va, vb, double(sgn[3 * int64_t(s) + a]), sb, k4, ik, lr, li);
#pragma unroll
                for (int b = 0; b < 3; ++b) {
                    if (NARROW && blk) {   // stored with the lower triangle as the row
                        const double *e = blk + 2 * (s <= t ? a * 3 + b : b * 3 + a);
                        lr[b] = e[0];
                        li[b] = e[1];
                    }
                    lr[b] = mine ? lr[b] : 0.0;
                    li[b] = mine ? li[b] : 0.0;
                }
#pragma unroll
                for (int i = 0; i < CI; ++i) {
                    const double c = cf[3 * i + a];
#pragma unroll
                    for (int b = 0; b < 3; ++b) {
                        double2 &z = sE[3 * i + b][tid];   // the lane's own
                        z.x += c * lr[b];
                        z.y += c * li[b];
                    }
                }
            }
        }
    }
    __syncthreads();
    const int32_t wf = max(w0, v);
    const int64_t hb = cells[wf].h0, nh = cells[w1 - 1].h0 + cells[w1 - 1].deg - hb;
    const int ni = min(CI, V.deg - i0);
    for (int64_t e = tid; e < nh * ni; e += CB) {
        const int i = int(e / nh);
        const int64_t h = hb + e % nh;
        const Cell W = cells[row_cell[h]];
        const int j = int(h - W.h0);
        double re = 0.0, im = 0.0;
        for (int u = 0; u < W.nt; ++u)
#pragma unroll
            for (int b = 0; b < 3; ++b) {
                const double c = coef[W.cf + (int64_t(u) * W.dp + j) * 3 + b];
                const double2 z = sE[3 * i + b][W.t0 - tb + u];
                re += c * z.x;
                im += c * z.y;
            }
        double2 *o = D + rowoff[V.h0 + i0 + i] + h;
        *o = NARROW ? make_double2(re, im) : make_double2(o->x + re, o->y + im);
    }
}

// T_BC(m, n) = sum over the rows h of m and h' of n (two ends, the parts of their
// cells) of D(h, h'), stored for h <= h'; hrow: rows of function m at hptr[m] ..
__global__ __launch_bounds__(CT) void k_cells_sum(int64_t n, const int32_t *__restrict__ hptr,
                                                  const int32_t *__restrict__ hrow, const int64_t *__restrict__ rowoff,
                                                  const double2 *__restrict__ D, double2 *__restrict__ T)
{
    const int64_t m = blockIdx.y, c = int64_t(blockIdx.x) * CT + threadIdx.x;
    if (c >= n) return;
    double re = 0.0, im = 0.0;
    for (int32_t a = hptr[m]; a < hptr[m + 1]; ++a) {
        const int64_t h = hrow[a];
        for (int32_t b = hptr[c]; b < hptr[c + 1]; ++b) {
            const int64_t g = hrow[b];
            const double2 z = D[h <= g ? rowoff[h] + g : rowoff[g] + h];
            re += z.x;
            im += z.y;
        }
    }
    T[m * n + c] = make_double2(re, im);
}

// ----------------------------------------------------------------------------- host geometry

struct V3 {
    double x, y, z;
};
inline V3 vsub(V3 a, V3 b) { return { a.x - b.x, a.y - b.y, a.z - b.z }; }
inline V3 vmid(V3 a, V3 b) { return { 0.5 * (a.x + b.x), 0.5 * (a.y + b.y), 0.5 * (a.z + b.z) }; }
inline V3 vcross(V3 a, V3 b) { return { a.y * b.z - a.z * b.y, a.z * b.x - a.x * b.z, a.x * b.y - a.y * b.x }; }
inline double vdot(V3 a, V3 b) { return a.x * b.x + a.y * b.y + a.z * b.z; }
inline V3 vscale(V3 a, double s) { return { a.x * s, a.y * s, a.z * s }; }

// Barycentric refinement of a validated closed mesh.
void refine(const Mesh &M, std::vector<double> &Vb, std::vector<int32_t> &Tb)
{
    const int64_t nv = M.nv, N = M.N, F = M.F;
    Vb.assign(3 * (nv + N + F), 0.0);
    std::copy(M.V.begin(), M.V.end(), Vb.begin());
    for (int64_t m = 0; m < N; ++m)
        for (int d = 0; d < 3; ++d)
            Vb[3 * (nv + m) + d] = 0.5 * (M.V[3 * M.edges[4 * m] + d] + M.V[3 * M.edges[4 * m + 1] + d]);
    for (int64_t t = 0; t < F; ++t)
        for (int d = 0; d < 3; ++d)
            Vb[3 * (nv + N + t) + d] =
                (M.V[3 * M.T[3 * t] + d] + M.V[3 * M.T[3 * t + 1] + d] + M.V[3 * M.T[3 * t + 2] + d]) / 3.0;
    Tb.assign(18 * F, 0);
    for (int64_t t = 0; t < F; ++t) {
        const int32_t g = int32_t(nv + N + t);
        for (int k = 0; k < 3; ++k) {
            const int32_t a = M.T[3 * t + k], b = M.T[3 * t + (k + 1) % 3];
            const int32_t mab = int32_t(nv + M.slot_m[3 * t + (k + 2) % 3]);   // edge a-b is opposite vertex k+2
            int32_t *c0 = &Tb[3 * (6 * t + 2 * k)];
            c0[0] = a; c0[1] = mab; c0[2] = g;
            c0[3] = mab; c0[4] = b; c0[5] = g;
        }
    }
}

// BC coefficients (CSR, N rows over the refined RWG functions) and the mixed Gram
// matrix (CSR, N x N) and its transpose.
void bc_and_gram(const Mesh &M, const Mesh &B, Csr &C, Csr &G, Csr &Gt)
{
    const int64_t N = M.N;
    // refined edge (v, mid) for the end v of m, or (mid, g) for v < 0, by triangle t's children at
    // edge m = a-b, 2k: (a, mid, g) and 2k + 1: (mid, b, g)
    auto child_edge = [&](int64_t m, int32_t t, int32_t v) {
        int k = 0;
        while (M.slot_m[3 * t + (k + 2) % 3] != m) ++k;
        const int64_t c = 6 * int64_t(t) + 2 * k;
        if (v < 0) return B.slot_m[3 * c];
        return B.slot_m[3 * (M.T[3 * t + k] == v ? c : c + 1) + 2];
    };
    auto sigma = [&](int32_t e, int32_t t) { return B.edges[4 * e + 2] == t ? 1.0 : -1.0; };
    auto across = [&](int32_t e, int32_t t) { return B.edges[4 * e + 2] == t ? B.edges[4 * e + 3] : B.edges[4 * e + 2]; };
    auto Vb = [&](int32_t v) { return V3{ B.V[3 * v], B.V[3 * v + 1], B.V[3 * v + 2] }; };
    // the radial edge of child t (corner v) other than e
    auto other_radial = [&](int32_t t, int32_t v, int32_t e) {
        int32_t out = -1;
        for (int k = 0; k < 3; ++k)
            if (B.T[3 * t + k] != v && B.slot_m[3 * t + k] != e) out = B.slot_m[3 * t + k];
        return out;
    };

    C.ptr.assign(1, 0);
    std::vector<std::pair<int32_t, double>> row;
    std::vector<int32_t> ts, es;
    for (int64_t m = 0; m < N; ++m) {
        row.clear();
        const int32_t lo = M.edges[4 * m], hi = M.edges[4 * m + 1], cp = M.edges[4 * m + 2], cm = M.edges[4 * m + 3];
        const int32_t half_p = child_edge(m, cp, -1), half_m = child_edge(m, cm, -1);
        for (int side = 0; side < 2; ++side) {
            const int32_t v = side == 0 ? hi : lo;
            const double charge = side == 0 ? 1.0 : -1.0;
            const int32_t e0 = child_edge(m, cp, v);
            const int32_t t1 = B.edges[4 * e0 + 2] / 6 == cp ? B.edges[4 * e0 + 2] : B.edges[4 * e0 + 3];
            ts.clear();
            es.clear();
            int32_t t = t1, prev = e0;
            while (true) {
                ts.push_back(t);
                const int32_t nx = other_radial(t, v, prev);
                if (nx == e0) break;
                es.push_back(nx);
                t = across(nx, t);
                prev = nx;
                if (ts.size() > 256) throw Error(BIE_EMESH, "dual cell walk did not close");
            }
            double Ac = 0.0;
            for (int32_t c : ts) Ac += B.area[c];
            double phi = 0.0;   // flux through the half of edge m: none
            for (size_t i = 0; i + 1 < ts.size(); ++i) {
                const double out_dual = i == 0 ? 0.5 * charge : 0.0;
                phi += charge * B.area[ts[i]] / Ac - out_dual;
                row.emplace_back(es[i], phi * sigma(es[i], ts[i]));
            }
            if (side == 0) {
                row.emplace_back(half_p, 0.5 * sigma(half_p, ts.front()));
                row.emplace_back(half_m, 0.5 * sigma(half_m, ts.back()));
            }
        }
        std::sort(row.begin(), row.end());
        for (auto &p : row) {
            C.idx.push_back(p.first);
            C.val.push_back(p.second);
        }
        C.ptr.push_back(int64_t(C.idx.size()));
    }

    // G_mn = <n x b_m, f_n>: first the integrals of every child's three refined functions
    // against its triangle's three
    std::vector<double> part(9 * size_t(B.F));
    for (int64_t T = 0; T < M.F; ++T) {
        const V3 p[3] = { { M.V[3 * M.T[3 * T]], M.V[3 * M.T[3 * T] + 1], M.V[3 * M.T[3 * T] + 2] },
                          { M.V[3 * M.T[3 * T + 1]], M.V[3 * M.T[3 * T + 1] + 1], M.V[3 * M.T[3 * T + 1] + 2] },
                          { M.V[3 * M.T[3 * T + 2]], M.V[3 * M.T[3 * T + 2] + 1], M.V[3 * M.T[3 * T + 2] + 2] } };
        V3 nrm = vcross(vsub(p[1], p[0]), vsub(p[2], p[0]));
        nrm = vscale(nrm, 1.0 / std::sqrt(vdot(nrm, nrm)));
        for (int64_t t = 6 * T; t < 6 * T + 6; ++t) {
            const V3 x[3] = { Vb(B.T[3 * t]), Vb(B.T[3 * t + 1]), Vb(B.T[3 * t + 2]) };
            const V3 xq[3] = { vmid(x[0], x[1]), vmid(x[1], x[2]), vmid(x[2], x[0]) };
            V3 f[3][3];   // function of slot sl at point q
            for (int sl = 0; sl < 3; ++sl) {
                const double sf = double(M.slot_s[3 * T + sl]) / (2.0 * M.area[T]);
                for (int q = 0; q < 3; ++q) f[sl][q] = vscale(vsub(xq[q], p[sl]), sf);
            }
            for (int a = 0; a < 3; ++a) {
                const double sb = double(B.slot_s[3 * t + a]) / (2.0 * B.area[t]);
                V3 rb[3];
                for (int q = 0; q < 3; ++q) rb[q] = vcross(nrm, vscale(vsub(xq[q], x[a]), sb));
                for (int sl = 0; sl < 3; ++sl) {
                    double sum = 0.0;
                    for (int q = 0; q < 3; ++q) sum += vdot(rb[q], f[sl][q]);
                    part[9 * t + 3 * a + sl] = sum;
                }
            }
        }
    }
    G.ptr.assign(1, 0);
    std::vector<double> acc(N, 0.0);
    std::vector<char> seen(N, 0);
    std::vector<int32_t> touched;
    for (int64_t m = 0; m < N; ++m) {
        touched.clear();
        for (int64_t k = C.ptr[m]; k < C.ptr[m + 1]; ++k) {
            const int32_t e = C.idx[k];
            const double ce = C.val[k];
            for (int side = 0; side < 2; ++side) {
                const int32_t t = B.edges[4 * e + 2 + side], T = t / 6;
                const int a = B.slot_m[3 * t] == e ? 0 : B.slot_m[3 * t + 1] == e ? 1 : 2;
                for (int sl = 0; sl < 3; ++sl) {
                    const int32_t n = M.slot_m[3 * T + sl];
                    if (!seen[n]) {
                        seen[n] = 1;
                        touched.push_back(n);
                    }
                    acc[n] += ce * B.area[t] / 3.0 * part[9 * size_t(t) + 3 * a + sl];
                }
            }
        }
        std::sort(touched.begin(), touched.end());
        for (int32_t n : touched) {
            G.idx.push_back(n);
            G.val.push_back(acc[n]);
            acc[n] = 0.0;
            seen[n] = 0;
        }
        G.ptr.push_back(int64_t(G.idx.size()));
    }
    // transpose
    Gt.ptr.assign(N + 1, 0);
    for (int32_t n : G.idx) Gt.ptr[n + 1] += 1;
    for (int64_t i = 0; i < N; ++i) Gt.ptr[i + 1] += Gt.ptr[i];
    Gt.idx.assign(G.idx.size(), 0);
    Gt.val.assign(G.val.size(), 0.0);
    std::vector<int64_t> fillp(Gt.ptr.begin(), Gt.ptr.end() - 1);
    for (int64_t m = 0; m < N; ++m)
        for (int64_t k = G.ptr[m]; k < G.ptr[m + 1]; ++k) {
            const int64_t d = fillp[G.idx[k]]++;
            Gt.idx[d] = int32_t(m);
            Gt.val[d] = G.val[k];
        }
}

// G X = B for the n columns of B by CG on the normal equations G^T G X = G^T B.
// R (input B, overwritten by the residual), X, P, W are n x n row-major (entry
// (i, c) at i n + c; column c is one right-hand side); sc holds 5 n + NSLICE n doubles.
constexpr int NSLICE = 64;

void gram_solve(const CsrDev &G, const CsrDev &Gt, int64_t n, double2 *Rr, double2 *X, double2 *P, double2 *W,
                double *sc, hipStream_t s, int64_t &iters, double &relres)
{
    const int64_t nn = n * n;
    double *zz = sc, *zn = sc + n, *ww = sc + 2 * n, *rr = sc + 3 * n, *bb = sc + 4 * n, *part = sc + 5 * n;
    const unsigned cb = unsigned((n + CT - 1) / CT);
    const dim3 mm(unsigned(n), cb);                               // sparse products: rows x column blocks
    const unsigned ew = unsigned(std::min<int64_t>((nn + CT - 1) / CT, 16384));
    auto colsq = [&](const double2 *A, double *out) {
        hipLaunchKernelGGL(k_colsq_part, dim3(cb, NSLICE), dim3(CT), 0, s, n, A, part);
        hipLaunchKernelGGL(k_colsq_fin, dim3(cb), dim3(CT), 0, s, n, NSLICE, (const double *)part, out);
    };
    hipLaunchKernelGGL(k_fill0, dim3(2048), dim3(256), 0, s, nn, X);
    colsq(Rr, bb);
    hipLaunchKernelGGL(k_csr_rm, mm, dim3(CT), 0, s, Gt.ptr, Gt.idx, Gt.val, n, Rr, P);   // z = G^T r
    colsq(P, zz);
    BIE_HIP(hipGetLastError());
    std::vector<double> hb(n), hr(n);
    BIE_HIP(hipMemcpyAsync(hb.data(), bb, n * sizeof(double), hipMemcpyDeviceToHost, s));
    BIE_HIP(hipStreamSynchronize(s));
    const double target = 1e-13;
    const int64_t maxit = 2000;
    relres = 1.0;
    for (iters = 1; iters <= maxit; ++iters) {
        hipLaunchKernelGGL(k_csr_rm, mm, dim3(CT), 0, s, G.ptr, G.idx, G.val, n, P, W);      // w = G p
        colsq(W, ww);
        hipLaunchKernelGGL(k_cg_xr, dim3(ew), dim3(CT), 0, s, n, zz, ww, P, W, X, Rr);
        hipLaunchKernelGGL(k_csr_rm, mm, dim3(CT), 0, s, Gt.ptr, Gt.idx, Gt.val, n, Rr, W);  // z = G^T r
        colsq(W, zn);
        hipLaunchKernelGGL(k_cg_p, dim3(ew), dim3(CT), 0, s, n, zn, zz, W, P);
        BIE_HIP(hipGetLastError());
        std::swap(zz, zn);
        if (iters % 8 == 0 || iters == maxit) {
            colsq(Rr, rr);
            BIE_HIP(hipMemcpyAsync(hr.data(), rr, n * sizeof(double), hipMemcpyDeviceToHost, s));
            BIE_HIP(hipStreamSynchronize(s));
            relres = 0.0;
            for (int64_t c = 0; c < n; ++c)
                if (hb[c] > 0.0) relres = std::max(relres, std::sqrt(hr[c] / hb[c]));
            if (relres <= target) break;
        }
    }
    if (relres > target) throw Error(BIE_ENUMERIC, "Gram solve of the Calderon preconditioner did not converge");
    iters = std::min(iters, maxit);
}

// G X = B by Chebyshev iteration on the interval [GA, GB] of the real axis (Saad,
// Iterative Methods for Sparse Linear Systems, Sec. 12.3).  The spectrum of the
// mixed Gram matrix lies in [1/3, 1) up to imaginary parts near 1e-3 on every mesh
// tried (spheres, ellipsoids up to 1:2:3, rounded cubes, area ratios up to 6):
// one sparse product per step and no inner products, about 0.3 per step.
constexpr double GA = 0.30, GB = 1.05;

// G in slices of 64 rows, entry e of a slice's rows side by side (width: the longest
// row; the others padded with zeros at their own column).
struct SlicedDev {
    int64_t rows = 0;
    int32_t *ptr = nullptr;    // first entry column of slice b; slices + 1
    uint16_t *idx = nullptr;   // [entry column][64]
    double *val = nullptr;
    void upload(const Csr &c)
    {
        rows = int64_t(c.ptr.size()) - 1;
        const int64_t ns = (rows + 63) / 64;
        std::vector<int32_t> p(1, 0);
        std::vector<uint16_t> ix;
        std::vector<double> vl;
        for (int64_t b = 0; b < ns; ++b) {
            int64_t w = 0;
            for (int64_t i = 64 * b; i < std::min(rows, 64 * b + 64); ++i) w = std::max(w, c.ptr[i + 1] - c.ptr[i]);
            const size_t at = vl.size();
            ix.resize(at + size_t(w) * 64, 0);
            vl.resize(at + size_t(w) * 64, 0.0);
            for (int64_t i = 64 * b; i < std::min(rows, 64 * b + 64); ++i)
                for (int64_t e = 0; e < w; ++e) {
                    const bool in = e < c.ptr[i + 1] - c.ptr[i];
                    ix[at + size_t(e * 64 + i - 64 * b)] = uint16_t(in ? c.idx[c.ptr[i] + e] : i);
                    if (in) vl[at + size_t(e * 64 + i - 64 * b)] = c.val[c.ptr[i] + e];
                }
            p.push_back(p.back() + int32_t(w));
        }
        BIE_HIP(device_malloc(&ptr, p.size() * sizeof(int32_t)));
        BIE_HIP(device_malloc(&idx, ix.size() * sizeof(uint16_t)));
        BIE_HIP(device_malloc(&val, vl.size() * sizeof(double)));
        BIE_HIP(hipMemcpy(ptr, p.data(), p.size() * sizeof(int32_t), hipMemcpyHostToDevice));
        BIE_HIP(hipMemcpy(idx, ix.data(), ix.size() * sizeof(uint16_t), hipMemcpyHostToDevice));
        BIE_HIP(hipMemcpy(val, vl.data(), vl.size() * sizeof(double), hipMemcpyHostToDevice));
    }
    ~SlicedDev()
    {
        if (ptr) (void)hipFree(ptr);
        if (idx) (void)hipFree(idx);
        if (val) (void)hipFree(val);
    }
};

// The columns are independent and G is real, so a block solves for NV real vectors
// by itself from the first step to the last: the direction D lies in LDS (the only
// array that neighbours read), X and the residual R in registers (rows tid,
// tid + 1024, ..., J of them), and nothing but G's 0.6 MB (L2) and the columns'
// first read and last write leaves the CU.  Steps over whole N x N blocks moved
// them through memory about ten times a step (2592 unknowns, 28 steps: 9.2 -> 1.95 ms).
// Column c of B is row c of the array Bt, column c of X row c of Xt.  NV = 2, 4, 8:
// NV / 2 complex columns; NV = 1: the real or the imaginary part of one.  The
// residual is checked every 4 steps; a block whose residual has not fallen by half
// since its last check (a spectrum outside the interval) reports failure.
struct GramStat {
    double relres;
    int32_t iters, ok;
};

template <int J, int NV>
__global__ __launch_bounds__(1024) void k_gram_cheb(int n, const int32_t *__restrict__ sptr,
                                                    const uint16_t *__restrict__ sidx, const double *__restrict__ sval,
                                                    const double *__restrict__ Bt, double *__restrict__ Xt,
                                                    GramStat *__restrict__ stat)
{
    constexpr int UN = NV >= 8 ? 1 : NV == 4 ? 2 : 4;   // entries in flight (registers)
    __shared__ double d[J * 1024 * NV];
    __shared__ double part[16][NV];
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const double theta = 0.5 * (GB + GA), delta = 0.5 * (GB - GA), sigma = theta / delta;
    // value v of row i: part v & 1 (or blockIdx & 1) of column c
    auto at = [&](int i, int v) -> int64_t {
        const int64_t c = NV == 1 ? blockIdx.x >> 1 : int64_t(blockIdx.x) * (NV / 2) + (v >> 1);
        return c < n && i < n ? 2 * (c * n + i) + (NV == 1 ? blockIdx.x & 1 : v & 1) : -1;
    };
    double x[J][NV], r[J][NV];
#pragma unroll
    for (int j = 0; j < J; ++j) {
        const int i = j * 1024 + tid;
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const int64_t o = at(i, v);
            r[j][v] = o >= 0 ? Bt[o] : 0.0;
            x[j][v] = 0.0;
            d[i * NV + v] = r[j][v] * (1.0 / theta);
        }
    }
    // sums of r^2 over the rows, in the same order for every lane
    auto squares = [&](double (&s)[NV]) {
        __syncthreads();
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            double a = 0.0;
#pragma unroll
            for (int j = 0; j < J; ++j) a += r[j][v] * r[j][v];
#pragma unroll
            for (int o = 32; o > 0; o >>= 1) a += __shfl_xor(a, o, 64);
            if (lane == 0) part[w][v] = a;
        }
        __syncthreads();
#pragma unroll
        for (int v = 0; v < NV; ++v) s[v] = 0.0;
#pragma unroll 1
        for (int u = 0; u < 16; ++u)
#pragma unroll
            for (int v = 0; v < NV; ++v) s[v] += part[u][v];
    };
    double bb[NV], rr[NV];
    squares(bb);
    double rho = 1.0 / sigma, last = 1.0, rel = 1.0;
    int it = 1, ok = 0;
    for (; it <= 200; ++it) {
        __syncthreads();   // D is written
#pragma unroll
        for (int j = 0; j < J; ++j) {
            const int b = j * 16 + w;   // slice of this wave's rows (uniform)
            if (64 * b >= n) break;
            double a[NV];
#pragma unroll
            for (int v = 0; v < NV; ++v) a[v] = 0.0;
            const int e1 = sptr[b + 1];
#pragma unroll UN
            for (int e = sptr[b]; e < e1; ++e) {
                const int k = sidx[e * 64 + lane];
                const double g = sval[e * 64 + lane];
#pragma unroll
                for (int v = 0; v < NV; ++v) a[v] += g * d[k * NV + v];
            }
#pragma unroll
            for (int v = 0; v < NV; ++v) r[j][v] -= a[v];
        }
        const double rhon = 1.0 / (2.0 * sigma - rho), c1 = rhon * rho, c2 = 2.0 * rhon / delta;
        rho = rhon;
        __syncthreads();   // D is read
#pragma unroll
        for (int j = 0; j < J; ++j)
#pragma unroll
            for (int v = 0; v < NV; ++v) {
                double &dd = d[(j * 1024 + tid) * NV + v];
                x[j][v] += dd;
                dd = c1 * dd + c2 * r[j][v];
            }
        if (it % 4) continue;
        squares(rr);
        rel = 0.0;
        bool finite = true;
#pragma unroll
        for (int v = 0; v < NV; ++v)
            if (bb[v] != 0.0) {   // a NaN column too
                const double q = sqrt(rr[v] / bb[v]);
                finite = finite && q < 1e300;
                rel = fmax(rel, q);
            }
        ok = finite && rel <= 1e-13;
        if (ok || !finite || !(rel < 0.5 * last)) break;
        last = rel;
    }
    if (tid == 0) stat[blockIdx.x] = { rel, it, ok };
#pragma unroll
    for (int j = 0; j < J; ++j)
#pragma unroll
        for (int v = 0; v < NV; ++v) {
            const int64_t o = at(j * 1024 + tid, v);
            if (o >= 0) Xt[o] = x[j][v];
        }
}

// Row c of Xt = G^{-1} (row c of Bt) for all n rows; false if a column failed.  NV:
// as many vectors as LDS (160 KB) and 128 registers a lane hold; each of them reads
// G once per step.
bool gram_solve_cheb(const SlicedDev &G, int64_t n, const double2 *Bt, double2 *Xt, hipStream_t s, int64_t &iters,
                     double &relres)
{
    const int64_t J = (n + 1023) / 1024;
    const int64_t nv = J <= 2 ? 8 : J <= 4 ? 4 : J <= 9 ? 2 : 1;
    const int64_t nblk = (2 * n + nv - 1) / nv;
    GramStat *ds = nullptr;
    BIE_HIP(device_malloc(&ds, size_t(nblk) * sizeof(GramStat)));
    std::vector<GramStat> h(nblk);
    auto run = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3(unsigned(nblk)), dim3(1024), 0, s, int(n), G.ptr, G.idx, G.val, (const double *)Bt,
                           (double *)Xt, ds);
    };
    switch (J) {
    case 1: run(k_gram_cheb<1, 8>); break;
    case 2: run(k_gram_cheb<2, 8>); break;
    case 3: run(k_gram_cheb<3, 4>); break;
    case 4: run(k_gram_cheb<4, 4>); break;
    case 5: run(k_gram_cheb<5, 2>); break;
    case 6: run(k_gram_cheb<6, 2>); break;
    case 7: run(k_gram_cheb<7, 2>); break;
    case 8: run(k_gram_cheb<8, 2>); break;
    case 9: run(k_gram_cheb<9, 2>); break;
    case 10: run(k_gram_cheb<10, 1>); break;
    case 11: run(k_gram_cheb<11, 1>); break;
    default: run(k_gram_cheb<12, 1>); break;   // CALDERON_MAX_N = 12 * 1024
    }
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) e = hipMemcpyAsync(h.data(), ds, h.size() * sizeof(GramStat), hipMemcpyDeviceToHost, s);
    const hipError_t e2 = hipStreamSynchronize(s);
    (void)hipFree(ds);
    BIE_HIP(e);
    BIE_HIP(e2);
    bool ok = true;
    iters = 0;
    relres = 0.0;
    for (const GramStat &g : h) {
        ok = ok && g.ok;
        iters = std::max<int64_t>(iters, g.iters);
        relres = std::max(relres, g.relres);
    }
    return ok;
}

void transpose(int64_t n, const double2 *A, double2 *B, hipStream_t s)
{
    hipLaunchKernelGGL(k_transpose, dim3(unsigned((n + 31) / 32), unsigned((n + 31) / 32)), dim3(32, 8), 0, s, n, A, B);
    BIE_HIP(hipGetLastError());
}

// Row c of Xt = G^{-1} (row c of Bt): Chebyshev, or CG on the normal equations if it
// fails (with BIE_CALDERON_GRAM=cgnr from the start).  Bt is kept.
void gram_solve_any(const SlicedDev &Gs, const Csr &G, const Csr &Gt, int64_t n, const double2 *Bt, double2 *Xt,
                    hipStream_t s, int64_t &iters, double &relres)
{
    const char *env = getenv("BIE_CALDERON_GRAM");
    const bool cg = env && std::string(env) == "cgnr";
    iters = 0;
    if (!cg && gram_solve_cheb(Gs, n, Bt, Xt, s, iters, relres)) return;
    CsrDev dG, dGt;
    dG.upload(G);
    dGt.upload(Gt);
    const size_t nn = size_t(n) * size_t(n);
    struct Work {
        void *p[4] = {};
        ~Work()
        {
            for (void *q : p)
                if (q) (void)hipFree(q);
        }
    } wk;
    for (int i = 0; i < 3; ++i) BIE_HIP(device_malloc(&wk.p[i], nn * sizeof(double2)));
    BIE_HIP(device_malloc(&wk.p[3], size_t((5 + NSLICE) * n) * sizeof(double)));
    double2 *Rr = static_cast<double2 *>(wk.p[0]), *X = static_cast<double2 *>(wk.p[1]),
            *P = static_cast<double2 *>(wk.p[2]);
    int64_t it2 = 0;
    transpose(n, Bt, Rr, s);
    gram_solve(dG, dGt, n, Rr, X, P, Xt, static_cast<double *>(wk.p[3]), s, it2, relres);   // Xt as its product array
    transpose(n, X, Xt, s);
    BIE_HIP(hipStreamSynchronize(s));
    iters += it2;
}

}  // namespace

// device copies of host tables, placed side by side and copied at once by send()
struct Bufs {
    std::vector<char> image;
    char *d = nullptr;
    ~Bufs()
    {
        if (d) (void)hipFree(d);
    }
    template <typename T>
    size_t add(const std::vector<T> &v)
    {
        const size_t at = (image.size() + 255) / 256 * 256;
        image.resize(at + v.size() * sizeof(T));
        if (!v.empty()) std::memcpy(image.data() + at, v.data(), v.size() * sizeof(T));
        return at;
    }
    void send()
    {
        BIE_HIP(device_malloc(&d, std::max<size_t>(1, image.size())));
        BIE_HIP(hipMemcpy(d, image.data(), image.size(), hipMemcpyHostToDevice));
    }
    template <typename T>
    const T *at(size_t o) const
    {
        return reinterpret_cast<const T *>(d + o);
    }
};

// T_BC (row-major n x n) of the BC functions C on the refined mesh of opb.
void dual_matrix(const Mesh &M, const bie_op *opb, const Csr &C, PoolBlock &work, double2 *T, hipStream_t s)
{
    const Mesh &B = opb->mesh;
    const TriDev &td = opb->tri;
    const int64_t N = M.N, Fb = B.F;
    const double near_factor = 2.0;   // the fill's default
    // edges of every vertex, and its children (the device order runs cell by cell)
    std::vector<int32_t> iptr(M.nv + 1, 0), inc(2 * N), place(2 * N);   // place: of edge m among its ends' edges
    for (int64_t i = 0; i < 2 * N; ++i) ++iptr[M.edges[4 * (i / 2) + i % 2] + 1];
    int32_t maxdeg = 1;
    for (int64_t v = 0; v < M.nv; ++v) {
        maxdeg = std::max(maxdeg, iptr[v + 1]);
        iptr[v + 1] += iptr[v];
    }
    {
        std::vector<int32_t> next(iptr.begin(), iptr.end() - 1);
        for (int64_t i = 0; i < 2 * N; ++i) {
            const int32_t v = M.edges[4 * (i / 2) + i % 2];
            place[i] = next[v] - iptr[v];
            inc[next[v]++] = int32_t(i / 2);
        }
    }
    const int ci = maxdeg <= 6 ? 6 : 8;
    std::vector<int32_t> tri_at(Fb), cell_of(Fb), cell_v, row_cell, row_m, group(1, 0), hptr(N + 1, 0);
    for (int64_t t = 0; t < Fb; ++t) tri_at[td.rank[t]] = int32_t(t);
    std::vector<Cell> cells;
    std::vector<double> longest(Fb);
    std::vector<int64_t> rowoff;
    int64_t ncoef = 0;
    int32_t r = 0, gchildren = 0;
    for (int64_t v = 0; v < M.nv; ++v) {
        const int32_t deg = iptr[v + 1] - iptr[v];
        int32_t left = 2 * deg;   // two children per triangle, a triangle per edge
        while (left > 0) {
            Cell c;
            c.t0 = r;
            c.nt = std::min(left, int32_t(CB));
            c.deg = deg;
            c.dp = (c.deg + ci - 1) / ci * ci;
            c.h0 = int64_t(row_cell.size());
            c.cf = ncoef;
            ncoef += int64_t(c.nt) * c.dp * 3;
            const int32_t id = int32_t(cells.size());
            if (gchildren + c.nt > CB) {
                group.push_back(id);
                gchildren = 0;
            }
            gchildren += c.nt;
            for (int32_t u = 0; u < c.nt; ++u) {
                const int32_t t = tri_at[r + u];
                if (B.T[3 * t] != v && B.T[3 * t + 1] != v) throw Error(BIE_EMESH, "refined triangles out of cell order");
                cell_of[r + u] = id;
                longest[r + u] = B.longest[t];
            }
            for (int32_t i = iptr[v]; i < iptr[v + 1]; ++i) {
                row_m.push_back(inc[i]);
                row_cell.push_back(id);
            }
            cells.push_back(c);
            cell_v.push_back(int32_t(v));
            r += c.nt;
            left -= c.nt;
        }
    }
    if (r != Fb) throw Error(BIE_EMESH, "dual cells do not cover the refined mesh");
    group.push_back(int32_t(cells.size()));
    const int64_t H = int64_t(row_cell.size());
    rowoff.resize(H);
    int64_t total = 0;
    for (int64_t h = 0; h < H; ++h) {   // row h: columns from its own cell's first on
        const int64_t c0 = cells[row_cell[h]].h0;
        rowoff[h] = total - c0;
        total += H - c0;
    }
    std::vector<int32_t> hrow(H);   // the rows of function m, in their order
    for (int64_t h = 0; h < H; ++h) ++hptr[row_m[h] + 1];
    for (int64_t m = 0; m < N; ++m) hptr[m + 1] += hptr[m];
    {
        std::vector<int32_t> next(hptr.begin(), hptr.end() - 1);
        for (int64_t h = 0; h < H; ++h) hrow[next[row_m[h]]++] = int32_t(h);
    }
    // the BC coefficients child by child: an edge of function m lies on two children of m's cells
    std::vector<double> coef(ncoef, 0.0);
    for (int64_t m = 0; m < N; ++m)
        for (int64_t k = C.ptr[m]; k < C.ptr[m + 1]; ++k)
            for (int side = 0; side < 2; ++side) {
                const int32_t e = C.idx[k], t = B.edges[4 * e + 2 + side], rt = td.rank[t], id = cell_of[rt];
                const Cell &c = cells[id];
                const int end = M.edges[4 * m] == cell_v[id] ? 0 : M.edges[4 * m + 1] == cell_v[id] ? 1 : -1;
                if (end < 0) continue;
                const int a = B.slot_m[3 * t] == e ? 0 : B.slot_m[3 * t + 1] == e ? 1 : 2;
                coef[c.cf + (int64_t(rt - c.t0) * c.dp + place[2 * m + end]) * 3 + a] = C.val[k];
            }
    work.get(std::max(size_t(total), 2 * size_t(N) * size_t(N)) * sizeof(double2));
    double2 *D = static_cast<double2 *>(work.p);
    double qwh[QPTS];
    quad_weights(qwh);

    NearDev nd;
    ranked_near(opb, near_factor, nd, s);
    Bufs bufs;
    const size_t o_c = bufs.add(cells), o_g = bufs.add(group), o_co = bufs.add(cell_of), o_rc = bufs.add(row_cell),
                 o_hp = bufs.add(hptr), o_hr = bufs.add(hrow), o_cf = bufs.add(coef), o_l = bufs.add(longest),
                 o_qw = bufs.add(std::vector<double>(qwh, qwh + QPTS)), o_ro = bufs.add(rowoff);
    bufs.send();
    const Cell *dc = bufs.at<Cell>(o_c);
    const int32_t *dg = bufs.at<int32_t>(o_g), *dco = bufs.at<int32_t>(o_co), *drc = bufs.at<int32_t>(o_rc),
                  *dhp = bufs.at<int32_t>(o_hp), *dhr = bufs.at<int32_t>(o_hr);
    const double *dcf = bufs.at<double>(o_cf), *dl = bufs.at<double>(o_l), *dqw = bufs.at<double>(o_qw);
    const int64_t *dro = bufs.at<int64_t>(o_ro);
    struct Pairs {
        int32_t *p = nullptr;
        ~Pairs()
        {
            if (p) (void)hipFree(p);
        }
    } pairs;
    pairs.p = near_list(nd, Fb, s);
    PoolBlock blocks(s);
    blocks.get(std::max<int64_t>(1, nd.n) * 18 * sizeof(double));
    double *fb = static_cast<double *>(blocks.p);
    singular_blocks(opb, pairs.p, nd.n, fb, s);
    const dim3 grid(unsigned(group.size() - 1), unsigned(cells.size()), unsigned((maxdeg + ci - 1) / ci));
    auto run = [&](auto kern) {
        hipLaunchKernelGGL(kern, grid, dim3(CB), 0, s, dc, dg, dco, drc, dcf, dro, td.cent, td.loc, td.vfree, td.sgn,
                           td.rad, dl, dqw, nd.ptr, nd.list, fb, near_factor, opb->k, D);
    };
    const bool wide = opb->k * 2.0 * td.max_rad > NARROW_PHASE;
    if (ci == 6) {
        run(k_cells<true, 6>);
        if (wide) run(k_cells<false, 6>);
    } else {
        run(k_cells<true, 8>);
        if (wide) run(k_cells<false, 8>);
    }
    hipLaunchKernelGGL(k_cells_sum, dim3(unsigned((N + CT - 1) / CT), unsigned(N)), dim3(CT), 0, s, N, dhp, dhr, dro,
                       (const double2 *)D, T);
    BIE_HIP(hipGetLastError());
    BIE_HIP(hipStreamSynchronize(s));
}

// Largest N for which the preconditioner is built (the rows a block of the Gram
// solves holds; its memory, 48 N^2 bytes of work arrays beside M, would allow more).
constexpr int64_t CALDERON_MAX_N = 12288;

bie_calderon *calderon_create(const bie_op *op, hipStream_t s)
{
    std::lock_guard<std::mutex> serial(g_setup_mu);
    const auto t0 = std::chrono::steady_clock::now();
    const Mesh &M = op->mesh;
    const int64_t N = M.N;
    if (N > CALDERON_MAX_N) throw Error(BIE_EINVAL, "Calderon preconditioner: N above 12288");
    if (op->star) throw Error(BIE_EINVAL, "Calderon preconditioner: needs an assembled operator");
    std::vector<double> Vb;
    std::vector<int32_t> Tb;
    refine(M, Vb, Tb);
    std::unique_ptr<bie_op, void (*)(bie_op *)> hold(new bie_op(), bie_op_destroy);
    bie_op *opb = hold.get();
    const int64_t Fb = int64_t(Tb.size() / 3);
    opb->mesh = build_mesh(Vb.data(), int64_t(Vb.size() / 3), Tb.data(), Fb, 2.0, false);   // pairs: ranked_near
    opb->device = op->device;
    opb->k = op->k;
    const int64_t Nb = opb->mesh.N;
    if (Nb != 9 * M.F) throw Error(BIE_EMESH, "refined mesh has an unexpected edge count");
    {
        // refined triangles cell by cell: child 2 i (2 i + 1) of a triangle lies at its corner i (i + 1)
        std::vector<int32_t> count(M.nv + 1, 0), order(Fb);
        auto corner = [&](int64_t t) { return M.T[3 * (t / 6) + (t % 6 / 2 + t % 2) % 3]; };
        for (int64_t t = 0; t < Fb; ++t) ++count[corner(t) + 1];
        for (int64_t v = 0; v < M.nv; ++v) count[v + 1] += count[v];
        for (int64_t t = 0; t < Fb; ++t) order[count[corner(t)]++] = int32_t(t);
        upload_triangles(opb, s, &order);
    }

    Csr C, G, Gt;
    bc_and_gram(M, opb->mesh, C, G, Gt);
    SlicedDev dG;
    dG.upload(G);

    std::unique_ptr<bie_calderon, void (*)(bie_calderon *)> pc(new bie_calderon(), calderon_destroy);
    pc->op = op;
    pc->info.N = N;
    pc->info.Nb = Nb;
    pc->info.nnz_bc = int64_t(C.idx.size());
    pc->info.nnz_gram = int64_t(G.idx.size());

    // T_BC, then A1^T = (G^{-1} T_BC)^T (T_BC symmetric: its columns are its rows),
    // A1, and M' = G^{-1} A1^T, transposed; M is symmetric, so either will do
    const int64_t nn = N * N;
    PoolBlock work(s), tbc(s);
    tbc.get(size_t(nn) * sizeof(double2));
    double2 *T = static_cast<double2 *>(tbc.p);
    dual_matrix(M, opb, C, work, T, s);
    hold.reset();   // the refined mesh is no longer needed
    double2 *X = static_cast<double2 *>(work.p), *Y = X + nn;
    gram_solve_any(dG, G, Gt, N, T, X, s, pc->info.cg_iters[0], pc->info.cg_relres[0]);
    transpose(N, X, Y, s);
    gram_solve_any(dG, G, Gt, N, Y, T, s, pc->info.cg_iters[1], pc->info.cg_relres[1]);

    // M = -(M' + M'^T)/2 in packed tiles
    bie_op *v = new bie_op();
    pc->view = v;
    v->device = op->device;
    v->k = op->k;
    v->storage = BIE_C128;
    v->mesh.N = N;
    packed_setup(v->pk, N, true);
    BIE_HIP(pool_get(&v->Z64, size_t(v->pk.ntiles) * TB * TB * sizeof(double2)));
    hipLaunchKernelGGL(k_pack_sym, dim3(unsigned(v->pk.nT), unsigned(v->pk.nT)), dim3(256), 0, s, N, v->pk.nT,
                       T, -1.0, (double2 *)v->Z64);
    BIE_HIP(hipGetLastError());
    BIE_HIP(hipStreamSynchronize(s));
    if (op->Abf) calderon_tm(pc.get(), s);   // block products of the preconditioned mixed solves
    pc->info.setup_ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
    return pc.release();
}

bie_op *calderon_tm(const bie_calderon *pcc, hipStream_t s)
{
    bie_calderon *pc = const_cast<bie_calderon *>(pcc);
    if (pc->tm) return pc->tm;
    const bie_op *op = pc->op;
    if (!op->Z64) throw Error(BIE_EINVAL, "Calderon preconditioner: T M needs the FP64 matrix");
    const int64_t N = pc->info.N, ch = std::min<int64_t>(N, 512);
    PoolBlock a(s), unit(s), prod(s);
    a.get(size_t(N) * N * sizeof(double2));
    unit.get(size_t(N) * ch * sizeof(double2));
    prod.get(size_t(N) * ch * sizeof(double2));
    double2 *A = static_cast<double2 *>(a.p), *I = static_cast<double2 *>(unit.p), *Mc = static_cast<double2 *>(prod.p);
    // column chunk of T M: unit vectors, M on the FP64 matrix cores, then T
    for (int64_t j0 = 0; j0 < N; j0 += ch) {
        const int64_t nc = std::min(ch, N - j0);
        hipLaunchKernelGGL(k_unit_cols, dim3(2048), dim3(256), 0, s, N, j0, nc, I);
        BIE_HIP(hipGetLastError());
        gemm64_product(pc->view, I, N, Mc, N, nullptr, 0, nc, nullptr, s);
        gemm64_product(op, Mc, N, A + j0 * N, N, nullptr, 0, nc, nullptr, s);
    }
    std::unique_ptr<bie_op, void (*)(bie_op *)> t(new bie_op(), bie_op_destroy);
    t->device = op->device;
    t->k = op->k;
    t->storage = BIE_SPLIT_BF16;
    t->mesh.N = N;
    split_dense(t.get(), A, s);   // synchronises
    pc->tm = t.release();
    return pc->tm;
}

void calderon_destroy(bie_calderon *pc)
{
    if (!pc) return;
    if (pc->view) bie_op_destroy(pc->view);   // every buffer the products made on it too
    if (pc->tm) bie_op_destroy(pc->tm);
    if (pc->tmp) (void)hipFree(pc->tmp);
    delete pc;
}

const bie_op *calderon_operator(const bie_calderon *pc) { return pc->op; }
const bie_calderon_info &calderon_info(const bie_calderon *pc) { return pc->info; }

// The operator holding M (packed FP64 tiles); split: also its split-BF16 copy for
// the block product (made on first use).
bie_op *calderon_view(const bie_calderon *pc, bool split, hipStream_t s)
{
    if (split && !pc->view->Abf) split_matrix(pc->view, s);
    return pc->view;
}

// The operator holding M with an FP32 copy of its packed tiles as well (made on
// first use, freed with the preconditioner), for products in FP32 storage.
bie_op *calderon_view32(const bie_calderon *pc, hipStream_t s)
{
    bie_op *v = pc->view;
    if (!v->Z32) {
        const int64_t n = v->pk.ntiles * TB * TB;
        void *z = nullptr;
        BIE_HIP(device_malloc(&z, size_t(n) * sizeof(float2)));
        convert_c128_to_c64(v->Z64, z, n, s);
        BIE_HIP(hipStreamSynchronize(s));
        v->Z32 = z;
    }
    return v;
}

// Two R x N complex128 scratch blocks for the preconditioned solve.
double2 *calderon_scratch(const bie_calderon *pcc, int64_t R, hipStream_t s)
{
    bie_calderon *pc = const_cast<bie_calderon *>(pcc);
    if (pc->tmp_R < R) {
        BIE_HIP(hipStreamSynchronize(s));
        if (pc->tmp) (void)hipFree(pc->tmp);
        pc->tmp = nullptr;
        pc->tmp_R = 0;
        BIE_HIP(device_malloc(&pc->tmp, size_t(2 * R * pc->info.N) * sizeof(double2)));
        pc->tmp_R = R;
    }
    return static_cast<double2 *>(pc->tmp);
}

void calderon_apply(const bie_calderon *pc, const void *X, int64_t ldx, void *Y, int64_t ldy, int64_t R,
                    const int *skip, int64_t sks, hipStream_t s)
{
    product(pc->view, MAT64, true, X, ldx, Y, ldy, nullptr, 0, R, skip, sks, false, s);
}

// x += a for n complex entries.
void add_into(int64_t n, const void *a, void *x, hipStream_t s)
{
    hipLaunchKernelGGL(k_add_cols, dim3(unsigned(std::min<int64_t>((n + 255) / 256, 4096))), dim3(256), 0, s, n,
                       (const double2 *)a, (double2 *)x);
    BIE_HIP(hipGetLastError());
}

void zero_into(int64_t n, void *x, hipStream_t s)
{
    hipLaunchKernelGGL(k_fill0, dim3(unsigned(std::min<int64_t>((n + 255) / 256, 4096))), dim3(256), 0, s, n,
                       (double2 *)x);
    BIE_HIP(hipGetLastError());
}

}  // namespace bie
