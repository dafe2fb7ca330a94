// Products with the dense impedance matrix in packed symmetric storage.
//
// The matrix-vector product is the O(N^2) operation of every Krylov
// iteration (Sec. I and II: dense storage and MVP cost).  The Galerkin EFIE
// matrix is symmetric (identical test and basis functions), and the fill makes
// it exactly so, which halves the bytes a product must stream: only the tiles
// (I, J), I <= J, of 64 x 64 entries are stored.  One pass over the tiles
// applies every off-diagonal tile twice,
//     y_I += T_IJ x_J     (row sums, kept in registers along a tile row)
//     y_J += T_IJ^T x_I   (column sums, one 64-entry partial per tile),
// and a second small kernel adds the partials of each 64-row block in a fixed
// order (deterministic, no atomics).
//
// Tile pass: one block of 4 waves walks a run of consecutive tiles of one tile
// row; wave w owns rows 16w..16w+15 of the row block, lane c owns column c.
// Every tile row (1 KiB in FP64) is read by one wave with one load per lane,
// 16 rows in flight per wave, and the next tile's loads are issued before the
// current tile's arithmetic.  Column sums of the 4 waves are combined through
// double-buffered LDS with one barrier per tile; x of the wave's 16 rows sits in
// scalar registers.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdlib>
#include <cstring>
#include <utility>
#include <mutex>
#include <string>
#include <vector>

#include "bie_internal.hpp"
#include "lanes.hpp"

namespace bie {

// Optional timing of the dense product kernels: events recorded on the launch
// stream around every launch (record 0: tile pass of the packed FP64/FP32
// product, 1: split-BF16 block product, 2: FP64 block product, 3: reduction of
// the packed product's partial sums, 4: block GMRES basis dots, 5: block GMRES
// basis update).
namespace prof {
bool on = false;
struct Rec {
    std::vector<std::pair<hipEvent_t, hipEvent_t>> ev;
    size_t used = 0;
    int64_t cols = 0;   // right-hand sides over the recorded launches
};
Rec rec[10];

void begin(int k, hipStream_t s, int64_t ncols)
{
    if (!on) return;
    Rec &r = rec[k];
    r.cols += ncols;
    if (r.used == r.ev.size()) {
        hipEvent_t a, b;
        BIE_HIP(hipEventCreate(&a));
        BIE_HIP(hipEventCreate(&b));
        r.ev.emplace_back(a, b);
    }
    BIE_HIP(hipEventRecord(r.ev[r.used].first, s));
}
void end(int k, hipStream_t s)
{
    if (!on) return;
    Rec &r = rec[k];
    BIE_HIP(hipEventRecord(r.ev[r.used].second, s));
    ++r.used;
}
}  // namespace prof

void prof_enable(bool enable) { prof::on = enable; }
bool prof_active() { return prof::on; }
void prof_begin(int kernel, hipStream_t s, int64_t ncols) { prof::begin(kernel, s, ncols); }
void prof_end(int kernel, hipStream_t s) { prof::end(kernel, s); }

void prof_read(int kernel, int64_t *launches, double *total_ms, int64_t *columns)
{
    if (kernel < 0 || kernel > 9) throw Error(BIE_EINVAL, "unknown kernel record");
    prof::Rec &r = prof::rec[kernel];
    double t = 0.0;
    for (size_t i = 0; i < r.used; ++i) {
        BIE_HIP(hipEventSynchronize(r.ev[i].second));
        float ms = 0.f;
        BIE_HIP(hipEventElapsedTime(&ms, r.ev[i].first, r.ev[i].second));
        t += ms;
    }
    *launches = int64_t(r.used);
    *total_ms = t;
    if (columns) *columns = r.cols;
    r.used = 0;
    r.cols = 0;
}

namespace {

// Tiles per unit of the single-operator tile pass, one unit per block, the same for any
// number of vectors (the units set the order of the sums).  Short units spread a small
// matrix over more CUs; long ones have fewer row sums and blocks, which is what many
// vectors ask for.  us, 1, 16 and 256 vectors (16 and 256: the better of the passes below):
//               FP64                                        FP32 matrix, FP64 vectors
//   unknowns    1 tile       2            4            8      1 tile       2           4
//     450       7  9  78     8  9  63     9 10  59    12 12   6  9  68     7  9  53    9 10  47
//     882       8 20 202     8 15 134    10 14 115    15 19   7 18 188     8 14 132   10 13 114
//    1152       8 30 313     9 23 222    12 22 179    14 20   7 27 302     8 20 216   10 19 173
//    1800      10 61 774    10 46 520    13 36 406    19 39   8 57 745     8 42 506   10 33 394
//    2592      16 112 1532  14 79 1026   15 66 797    20 58  12 107 1473  11 75 994   11 62 769
//    4608      39 328       36 219       37 171       36 156  28 310      25 209      24 162
//    7680      98 960       90 635       87 496       88 454  67 880      53 582      47 443
// (8 against 16 tiles, one FP64 vector: 115 / 127 at 8712, 185 / 193 at 11250).  A unit of one
// tile gains one vector under 1 us over two and costs 128 and more up to a third.
// BIE_SYM_UNIT = 1..64 fixes the length, 0 balanced runs (measurement).
int unit_tiles(int64_t nT, bool mat64)
{
    static const int env = [] {
        const char *e = getenv("BIE_SYM_UNIT");
        const int u = e ? atoi(e) : -1;
        return e ? (u >= 0 && u <= 64 ? u : 8) : -1;
    }();
    if (env >= 0) return env;
    const int64_t tiles = nT * (nT + 1) / 2;
    return tiles < (mat64 ? 600 : 150) ? 2 : tiles < 3072 ? 4 : 8;
}

typedef double nd2 __attribute__((ext_vector_type(2)));
typedef float nf2 __attribute__((ext_vector_type(2)));

template <typename T>
struct Cx;   // complex element as a native 2-vector (one load instruction)
template <>
struct Cx<double> {
    using type = nd2;
};
template <>
struct Cx<float> {
    using type = nf2;
};

__device__ __forceinline__ double fma_(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ __forceinline__ float fma_(float a, float b, float c) { return __builtin_fmaf(a, b, c); }

// (ar, ai) += z x, in the one order that every tile pass uses
template <typename T>
__device__ __forceinline__ void cmad(T &ar, T &ai, T zr, T zi, T xr, T xi)
{
    ar = fma_(zr, xr, ar);
    ar = fma_(-zi, xi, ar);
    ai = fma_(zr, xi, ai);
    ai = fma_(zi, xr, ai);
}

template <typename T>
__device__ inline T wsum(T v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

// Tile pass of one work unit: tiles (I, J0 .. J1-1) of row block I, the
// unit being the uo-th of its row.  Writes 64-entry partial vectors (complex
// T) into the slots of the row block they belong to (see reduce_rows).
// M: matrix storage type, T: vector and accumulation type (T >= M).  NT:
// non-temporal tile loads (one vector streams the matrix once; several
// vectors re-read the unit's tiles from the caches).
template <typename M, typename T, bool CONJ, bool PREFETCH, bool NT = true>
__device__ __forceinline__ void tile_pass(const M *__restrict__ Zp, int64_t N, int64_t nT, int32_t I, int32_t J0, int32_t J1,
                                 int64_t uo, const int64_t *__restrict__ seg,
                                 const typename Cx<T>::type *__restrict__ x, typename Cx<T>::type *__restrict__ pv)
{
    using V2 = typename Cx<T>::type;
    using MV = typename Cx<M>::type;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // uniform: x rows in scalar registers
    // partials of row block K live in slots seg[K]..: first the column sums of
    // tiles (0..K-1, K), then the row sums of the units of tile row K
    const MV *Z = reinterpret_cast<const MV *>(Zp);

    // x of this wave's 16 rows (the same for every lane)
    T xir[16], xii[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
        const int64_t m = int64_t(I) * TB + wave * 16 + i;
        V2 xv = { 0, 0 };
        if (m < N) xv = x[m];
        xir[i] = xv.x;
        xii[i] = xv.y;
    }
    T rar[16], rai[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) { rar[i] = 0; rai[i] = 0; }
    __shared__ V2 red[2][8][TB];

    // x_J of lane's column, loaded with the tile it multiplies (a load issued
    // just before its use would expose its latency once per tile)
    auto xcol = [&](int32_t J) {
        const int64_t n = int64_t(J) * TB + lane;
        V2 v = { 0, 0 };
        if (n < N) v = x[n];
        return v;
    };
    MV t[16];
    V2 xt = { 0, 0 };
    if (PREFETCH) {
        const MV *tile = Z + tile_of(I, J0, nT) * TB * TB + (wave * 16) * TB + lane;
#pragma unroll
        for (int i = 0; i < 16; ++i) t[i] = NT ? __builtin_nontemporal_load(tile + i * TB) : tile[i * TB];
        xt = xcol(J0);
    }
    for (int32_t J = J0; J < J1; ++J) {
        V2 xj;
        MV cur[16];
        if (PREFETCH) {
#pragma unroll
            for (int i = 0; i < 16; ++i) cur[i] = t[i];
            xj = xt;
            if (J + 1 < J1) {   // next tile's loads go out before this tile's arithmetic
                const MV *tile = Z + tile_of(I, J + 1, nT) * TB * TB + (wave * 16) * TB + lane;
#pragma unroll
                for (int i = 0; i < 16; ++i) t[i] = NT ? __builtin_nontemporal_load(tile + i * TB) : tile[i * TB];
                xt = xcol(J + 1);
            }
        } else {
            xj = xcol(J);
            const MV *tile = Z + tile_of(I, J, nT) * TB * TB + (wave * 16) * TB + lane;
#pragma unroll
            for (int i = 0; i < 16; ++i) cur[i] = NT ? __builtin_nontemporal_load(tile + i * TB) : tile[i * TB];
        }
        // column sums by groups of 8 rows (the rows of a wave of the several-vector
        // pass, whose columns equal this pass's bit for bit)
        T car[2] = { 0, 0 }, cai[2] = { 0, 0 };
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const T zr = T(cur[i].x), zi = CONJ ? -T(cur[i].y) : T(cur[i].y);
            cmad(rar[i], rai[i], zr, zi, xj.x, xj.y);
            cmad(car[i >> 3], cai[i >> 3], zr, zi, xir[i], xii[i]);
        }
        if (J != I) {   // uniform over the block
            // double-buffered by tile parity: one barrier per tile; the barrier of
            // the next tile orders this tile's reads before the buffer is reused
            const int par = (J - J0) & 1;
            red[par][2 * wave][lane] = V2{ car[0], cai[0] };
            red[par][2 * wave + 1][lane] = V2{ car[1], cai[1] };
            __syncthreads();
            if (wave == ((J - J0) & 3)) {
                V2 a = red[par][0][lane];
#pragma unroll
                for (int w = 1; w < 8; ++w) a += red[par][w][lane];
                pv[(seg[J] + I) * TB + lane] = a;
            }
        }
    }
    // row sums: 16 values per wave, two groups of 8
#pragma unroll
    for (int g = 0; g < 2; ++g) {
        T pr[8], pi[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) { pr[i] = rar[8 * g + i]; pi[i] = rai[8 * g + i]; }
        wave_sum8(pr, pi);
        if ((lane & 7) == 0) pv[(seg[I] + I + uo) * TB + wave * 16 + 8 * g + (lane >> 3)] = V2{ pr[0], pi[0] };
    }
}

// Tile pass over the units of one problem: block (run b, vector v) takes the
// units run_ptr[b] .. run_ptr[b+1]-1 in turn (a barrier between units: the
// LDS buffers of the column sums restart at parity 0).  At most 256 VGPRs:
// two blocks per CU.
template <typename M, typename T, bool CONJ, bool PREFETCH, bool NT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_sym_tiles(const M *__restrict__ Zp, int64_t N, int64_t nT,
                                                   const int32_t *__restrict__ units,
                                                   const int32_t *__restrict__ unit_ptr,
                                                   const int32_t *__restrict__ run_ptr,
                                                   const int64_t *__restrict__ seg, int64_t nslots,
                                                   const T *__restrict__ X, int64_t ldx, T *__restrict__ part,
                                                   const int *__restrict__ skip, int64_t sks)
{
    using V2 = typename Cx<T>::type;
    const int64_t v = blockIdx.y;
    if (skip && skip[v * sks]) return;
    const int32_t u0 = run_ptr[blockIdx.x], u1 = run_ptr[blockIdx.x + 1];
    for (int32_t u = u0; u < u1; ++u) {
        if (u > u0) __syncthreads();
        const int32_t I = units[3 * u], J0 = units[3 * u + 1], J1 = units[3 * u + 2];
        tile_pass<M, T, CONJ, PREFETCH, NT>(Zp, N, nT, I, J0, J1, u - unit_ptr[I], seg,
                                        reinterpret_cast<const V2 *>(X) + v * ldx,
                                        reinterpret_cast<V2 *>(part) + v * nslots * TB);
    }
}

// The same for several vectors: a block of 8 waves takes a run for NC of them at
// once, each wave 8 rows of the row block, so that a tile read serves NC products
// (one block per vector read the matrix R times: 6 FP64 vectors at 5202 unknowns
// 237 -> 80 us, 16 at 7680 1307 -> 454 us).  The row sums of NC vectors fill the registers (2 waves per SIMD at
// NC = 3); x of the tile rows comes from LDS, the same address for every lane.  The
// groups of one run start together on one XCD, so that its L2 serves all but one of
// them.  NT: as in the single-vector pass.  Every column has the bits of a product
// of its own.
template <typename M, typename T, bool CONJ, int NC, bool NT>
__global__ __launch_bounds__(512) void k_sym_tiles_n(int nruns, const M *__restrict__ Zp, int64_t N, int64_t nT,
                                                     const int32_t *__restrict__ units,
                                                     const int32_t *__restrict__ unit_ptr,
                                                     const int32_t *__restrict__ run_ptr,
                                                     const int64_t *__restrict__ seg, int64_t nslots, int G, int64_t R,
                                                     const T *__restrict__ Xp, int64_t ldx, T *__restrict__ part,
                                                     const int *__restrict__ skip, int64_t sks)
{
    using V2 = typename Cx<T>::type;
    using MV = typename Cx<M>::type;
    __shared__ V2 red[2][NC][8][TB];
    __shared__ V2 sx[TB][NC];
    // consecutive blocks go to the 8 XCDs in turn: the G groups of a run are 8 apart
    const int r8 = blockIdx.x % (8 * G);
    const int32_t run = blockIdx.x / (8 * G) * 8 + r8 % 8;
    if (run >= nruns) return;
    const int64_t c0 = int64_t(r8 / 8) * NC;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    bool live[NC], any = false;   // uniform; columns beyond R repeat the last one and store nothing
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        live[c] = c0 + c < R && !(skip && skip[(c0 + c) * sks]);
        any = any || live[c];
    }
    if (!any) return;
    const V2 *x[NC];
    V2 *pv[NC];
#pragma unroll
    for (int c = 0; c < NC; ++c) {
        const int64_t col = c0 + c < R ? c0 + c : R - 1;
        x[c] = reinterpret_cast<const V2 *>(Xp) + col * ldx;
        pv[c] = reinterpret_cast<V2 *>(part) + col * nslots * TB;
    }
    const MV *Z = reinterpret_cast<const MV *>(Zp);
    for (int32_t u = run_ptr[run]; u < run_ptr[run + 1]; ++u) {
        const int32_t I = units[3 * u], J0 = units[3 * u + 1], J1 = units[3 * u + 2];
        __syncthreads();   // the previous unit's LDS reads are done
        for (int e = threadIdx.x; e < TB * NC; e += 512) {
            const int64_t m = int64_t(I) * TB + e / NC;
            V2 v = { 0, 0 };
#pragma unroll
            for (int c = 0; c < NC; ++c)
                if (e % NC == c && m < N) v = x[c][m];
            sx[e / NC][e % NC] = v;
        }
        __syncthreads();
        T rar[8][NC], rai[8][NC];
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int c = 0; c < NC; ++c) rar[i][c] = rai[i][c] = 0;
        MV t[8];
        const auto load = [&](int32_t J) {
            const MV *tile = Z + tile_of(I, J, nT) * TB * TB + (wave * 8) * TB + lane;
#pragma unroll
            for (int i = 0; i < 8; ++i) t[i] = NT ? __builtin_nontemporal_load(tile + i * TB) : tile[i * TB];
        };
        load(J0);
        for (int32_t J = J0; J < J1; ++J) {
            asm volatile("" ::: "memory");   // x of the tile rows is read from LDS for every tile: no registers for it
            MV cur[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) cur[i] = t[i];
            V2 xj[NC];
            const int64_t n = int64_t(J) * TB + lane;
#pragma unroll
            for (int c = 0; c < NC; ++c) {
                xj[c] = V2{ 0, 0 };
                if (n < N) xj[c] = x[c][n];
            }
            if (J + 1 < J1) load(J + 1);
            T car[NC], cai[NC];
#pragma unroll
            for (int c = 0; c < NC; ++c) car[c] = cai[c] = 0;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const T zr = T(cur[i].x), zi = CONJ ? -T(cur[i].y) : T(cur[i].y);
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    const V2 xi = sx[wave * 8 + i][c];
                    cmad(rar[i][c], rai[i][c], zr, zi, xj[c].x, xj[c].y);
                    cmad(car[c], cai[c], zr, zi, xi.x, xi.y);
                }
            }
            if (J != I) {   // uniform over the block
                const int par = (J - J0) & 1;
#pragma unroll
                for (int c = 0; c < NC; ++c) red[par][c][wave][lane] = V2{ car[c], cai[c] };
                __syncthreads();
#pragma unroll
                for (int c = 0; c < NC; ++c)
                    if (wave == ((J - J0 + c) & 7) && live[c]) {
                        V2 a = red[par][c][0][lane];
#pragma unroll
                        for (int w = 1; w < 8; ++w) a += red[par][c][w][lane];
                        pv[c][(seg[J] + I) * TB + lane] = a;
                    }
            }
        }
#pragma unroll
        for (int c = 0; c < NC; ++c) {
            T pr[8], pi[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) { pr[i] = rar[i][c]; pi[i] = rai[i][c]; }
            wave_sum8(pr, pi);
            if ((lane & 7) == 0 && live[c])
                pv[c][(seg[I] + I + u - unit_ptr[I]) * TB + wave * 8 + (lane >> 3)] = V2{ pr[0], pi[0] };
        }
    }
}

// a value known to be the same in every lane, moved to scalar registers
__device__ inline int64_t uniform64(int64_t v)
{
    const uint64_t u = uint64_t(v);
    const uint32_t lo = __builtin_amdgcn_readfirstlane(uint32_t(u)), hi = __builtin_amdgcn_readfirstlane(uint32_t(u >> 32));
    return int64_t((uint64_t(hi) << 32) | lo);
}

// Grouped tile pass over several problems: block b is the work item (problem
// p, unit u, column group g) and goes through columns c0 + gG .. of p in turn,
// skipping finished ones; the unit's tiles come from memory for the first
// column and from the caches for the others.  A barrier separates the columns:
// the column-sum buffers of the tile pass start again at parity 0, and the
// last tile's buffer may still be read by another wave.  Items are ordered
// longest first.
template <typename M, typename T, bool PREFETCH>
__global__ __launch_bounds__(256) void k_sym_tiles_g(const GProb *__restrict__ probs, GCols gc,
                                                     const int32_t *__restrict__ items, int G, const T *__restrict__ X,
                                                     T *__restrict__ part, const int *__restrict__ skip, int64_t sks)
{
    using V2 = typename Cx<T>::type;
    const int64_t b = blockIdx.x;
    const int32_t p = items[3 * b], u = items[3 * b + 1], g = items[3 * b + 2];
    const GProb P = probs[p];
    // values read through the tables' pointers are the same in every lane:
    // made scalar so that the tile pass keeps its row indices and x of the
    // tile rows in scalar registers, as in the single-operator pass
    const int32_t I = __builtin_amdgcn_readfirstlane(P.units[3 * u]);
    const int32_t J0 = __builtin_amdgcn_readfirstlane(P.units[3 * u + 1]);
    const int32_t J1 = __builtin_amdgcn_readfirstlane(P.units[3 * u + 2]);
    const int32_t uo = __builtin_amdgcn_readfirstlane(u - P.unit_ptr[I]);
    const int32_t cb = P.c0 + g * G, ce = min(P.c1, cb + G);
    bool first = true;
    for (int32_t c = cb; c < ce; ++c) {
        if (skip && skip[int64_t(c) * sks]) continue;   // uniform over the block
        if (!first) __syncthreads();
        first = false;
        const int64_t xo = uniform64(gc.xoff[c] + gc.xstep * P.N), po = uniform64(gc.poff[c] * TB);
        tile_pass<M, T, false, PREFETCH, false>(static_cast<const M *>(P.Z), P.N, P.nT, I, J0, J1, uo, P.seg,
                                                reinterpret_cast<const V2 *>(X) + xo,
                                                reinterpret_cast<V2 *>(part) + po);
    }
}

// Grouped tile pass on the FP32 matrix cores (batches certified by FP64
// residuals): block b is the work item (problem p, unit u, column group g of
// at most 32 columns, padded with zeros to 32).  Per tile (I, J) of the unit
// the complex products Y_I += Z X_J (rows of block I, accumulated over the
// unit) and, for J != I, Y_J = Z^T X_I (written per tile) are four real
// 32 x 32 x 2 chains of v_mfma_f32_32x32x2f32 per wave: wave w = 2 h + part
// computes rows (or tile columns) 32 h .. 32 h + 31 of the real (part 0) or the
// imaginary (part 1) output.  The tile (rows padded to 65 entries) and the two
// vector blocks are staged in LDS in FP32 (the vectors rounded from FP64);
// accumulation is FP32 within the unit; the partial vectors go to the same
// FP64 slots as the VALU tile pass's, so the same reduction sums them.
typedef float f32x16g __attribute__((ext_vector_type(16)));
typedef float f32x4g __attribute__((ext_vector_type(4)));
// Loads that name the global address space.  Pointers read from the problem
// table are generic, and a generic (flat) load also counts against the LDS wait
// counter: the waits for the LDS fragment reads would then wait for the next
// tile's prefetch as well.
typedef float gf2v __attribute__((ext_vector_type(2)));
typedef double gd2v __attribute__((ext_vector_type(2)));
__device__ inline float2 gload_f2(const float2 *p, int64_t i)
{
    const gf2v v = ((const __attribute__((address_space(1))) gf2v *)p)[i];
    return make_float2(v[0], v[1]);
}
__device__ inline double2 gload_d2(const double2 *p, int64_t i)
{
    const gd2v v = ((const __attribute__((address_space(1))) gd2v *)p)[i];
    return make_double2(v[0], v[1]);
}
__device__ inline int64_t gload_i64(const int64_t *p, int64_t i)
{
    return ((const __attribute__((address_space(1))) int64_t *)p)[i];
}

__global__ __launch_bounds__(256) void k_sym_tiles_gm(const GProb *__restrict__ probs, GCols gc,
                                                      const int32_t *__restrict__ items, int G,
                                                      const double *__restrict__ X, float *__restrict__ part,
                                                      const int *__restrict__ skip, int64_t sks)
{
    __shared__ float2 sZ[TB][TB + 1];
    __shared__ float2 sXI[TB][32];
    __shared__ float2 sXJ[TB][32];
    __shared__ int32_t live[32];
    const int64_t b = blockIdx.x;
    const int32_t p = items[3 * b], u = items[3 * b + 1], g = items[3 * b + 2];
    const GProb P = probs[p];
    const int32_t I = __builtin_amdgcn_readfirstlane(P.units[3 * u]);
    const int32_t J0 = __builtin_amdgcn_readfirstlane(P.units[3 * u + 1]);
    const int32_t J1 = __builtin_amdgcn_readfirstlane(P.units[3 * u + 2]);
    const int32_t uo = __builtin_amdgcn_readfirstlane(u - P.unit_ptr[I]);
    const int32_t cb = P.c0 + g * G, ce = min(min(P.c1, cb + G), cb + 32);
    const int nc = ce - cb;
    const int t = threadIdx.x, lane = t & 63, w = t >> 6, h = w >> 1, prt = w & 1, li = lane & 31, lk = lane >> 5;
    if (t < 32) live[t] = (t < nc && !(skip && skip[int64_t(cb + t) * sks])) ? 1 : 0;
    __syncthreads();
    int hi = 0;   // one past the last live column
    for (int c = 0; c < nc; ++c)
        if (live[c]) hi = c + 1;
    if (hi == 0) return;   // uniform over the block
    // at most 16 live leading columns: 16 x 16 products (half the matrix-core work)
    const bool narrow = hi <= 16;
    const float2 *Z = static_cast<const float2 *>(P.Z);
    const double2 *Xc = reinterpret_cast<const double2 *>(X);
    // staging: thread t always moves column t & 31 of the vectors (rows t/32 + 8 i)
    // and entries t + 256 i of the tile (row t/64 + 4 i, column t & 63)
    const int sc = t & 31, sr = t >> 5;
    const bool slive = live[sc] != 0;
    const int64_t sxo = slive ? gc.xoff[cb + sc] + gc.xstep * P.N : 0;
    auto load_x = [&](double2 (&xv)[8], int32_t blk) {
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int64_t row = int64_t(blk) * TB + sr + 8 * q;
            xv[q] = (slive && row < P.N) ? gload_d2(Xc, sxo + row) : make_double2(0.0, 0.0);
        }
    };
    auto put_x = [&](float2 (*dst)[32], const double2 (&xv)[8]) {
#pragma unroll
        for (int q = 0; q < 8; ++q) dst[sr + 8 * q][sc] = make_float2(float(xv[q].x), float(xv[q].y));
    };
    auto load_z = [&](float2 (&zv)[16], int32_t J) {
        const float2 *tile = Z + tile_of(I, J, P.nT) * TB * TB + t;
#pragma unroll
        for (int q = 0; q < 16; ++q) zv[q] = gload_f2(tile, 256 * q);
    };
    auto put_z = [&](const float2 (&zv)[16]) {
#pragma unroll
        for (int q = 0; q < 16; ++q) sZ[(t >> 6) + 4 * q][t & 63] = zv[q];
    };
    // one real 32 x 32 output of the complex product over the 64 entries of k
    auto chain = [&](f32x16g acc, bool transposed, float2 (*xs)[32]) {
#pragma unroll 8
        for (int k0 = 0; k0 < TB; k0 += 2) {
            const float2 z = transposed ? sZ[k0 + lk][32 * h + li] : sZ[32 * h + li][k0 + lk];
            const float2 x = xs[k0 + lk][li];
            if (prt == 0) {
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(z.x, x.x, acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(-z.y, x.y, acc, 0, 0, 0);
            } else {
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(z.x, x.y, acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(z.y, x.x, acc, 0, 0, 0);
            }
        }
        return acc;
    };
    // value q of lane l: row 32 h + 8 (q / 4) + 4 (l / 32) + q % 4, column l % 32
    const bool olive = live[li] != 0;
    const int64_t opo = olive ? gc.poff[cb + li] * TB : 0;
    auto store = [&](const f32x16g &acc, int64_t slot) {
        if (!olive) return;
        float *pv = part + (opo + slot * TB) * 2 + prt;
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const int r = 32 * h + 8 * (q >> 2) + 4 * lk + (q & 3);
            pv[2 * r] = acc[q];
        }
    };
    // narrow form: wave w takes rows 16 w .. + 15 of the tile and both parts;
    // v_mfma_f32_16x16x4f32: A[i][k] in lane i + 16 k, B[k][j] in lane j + 16 k,
    // output value q of lane l at row 4 (l / 16) + q, column l % 16
    const int ni = lane & 15, nk = lane >> 4;
    auto chain16 = [&](f32x4g &ar, f32x4g &ai, bool transposed, float2 (*xs)[32]) {
#pragma unroll 4
        for (int k0 = 0; k0 < TB; k0 += 4) {
            const float2 z = transposed ? sZ[k0 + nk][16 * w + ni] : sZ[16 * w + ni][k0 + nk];
            const float2 x = xs[k0 + nk][ni];
            ar = __builtin_amdgcn_mfma_f32_16x16x4f32(z.x, x.x, ar, 0, 0, 0);
            ar = __builtin_amdgcn_mfma_f32_16x16x4f32(-z.y, x.y, ar, 0, 0, 0);
            ai = __builtin_amdgcn_mfma_f32_16x16x4f32(z.x, x.y, ai, 0, 0, 0);
            ai = __builtin_amdgcn_mfma_f32_16x16x4f32(z.y, x.x, ai, 0, 0, 0);
        }
    };
    const bool nlive = live[ni] != 0;
    const int64_t npo = nlive ? gc.poff[cb + ni] * TB : 0;
    auto store16 = [&](const f32x4g &ar, const f32x4g &ai, int64_t slot) {
        if (!nlive) return;
        float *pv = part + (npo + slot * TB) * 2;
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int r = 16 * w + 4 * nk + q;
            pv[2 * r] = ar[q];
            pv[2 * r + 1] = ai[q];
        }
    };
    double2 xv[8];
    float2 zv[16];
    load_x(xv, I);
    put_x(sXI, xv);
    load_z(zv, J0);
    load_x(xv, J0);
    f32x16g arow;
    f32x4g nrr, nri;
#pragma unroll
    for (int q = 0; q < 16; ++q) arow[q] = 0.f;
#pragma unroll
    for (int q = 0; q < 4; ++q) nrr[q] = nri[q] = 0.f;
    for (int32_t J = J0; J < J1; ++J) {
        __syncthreads();   // the previous tile's LDS reads are done
        put_z(zv);
        put_x(sXJ, xv);
        __syncthreads();
        if (J + 1 < J1) {   // the next tile's loads go out before this tile's products
            load_z(zv, J + 1);
            load_x(xv, J + 1);
        }
        if (narrow) {
            chain16(nrr, nri, false, sXJ);
            if (J != I) {
                f32x4g cr, ci;
#pragma unroll
                for (int q = 0; q < 4; ++q) cr[q] = ci[q] = 0.f;
                chain16(cr, ci, true, sXI);
                store16(cr, ci, gload_i64(P.seg, J) + I);
            }
        } else {
            arow = chain(arow, false, sXJ);
            if (J != I) {
                f32x16g acol;
#pragma unroll
                for (int q = 0; q < 16; ++q) acol[q] = 0.f;
                acol = chain(acol, true, sXI);
                store(acol, gload_i64(P.seg, J) + I);
            }
        }
    }
    if (narrow) store16(nrr, nri, gload_i64(P.seg, I) + I + uo);
    else store(arow, gload_i64(P.seg, I) + I + uo);
}

// The same grouped pass on FP64 tiles with the FP64 matrix cores
// (v_mfma_f64_16x16x4f64: A[i][k] in lane i + 16 k, B[k][j] in lane j + 16 k,
// output value q of lane l at row l / 16 + 4 q, column l % 16 -- rows
// interleaved, unlike the FP32 16 x 16 x 4 form): wave w takes
// rows 16 w .. + 15 of the tile, both parts, and the item's columns in halves of
// 16 (one half when the live columns fit in it).  The tile (64 KB) and the two
// vector blocks stay FP64 in LDS; FP64 accumulation throughout.
typedef double f64x4g __attribute__((ext_vector_type(4)));

__global__ __launch_bounds__(256) void k_sym_tiles_gm64(const GProb *__restrict__ probs, GCols gc,
                                                        const int32_t *__restrict__ items, int G,
                                                        const double *__restrict__ X, double *__restrict__ part,
                                                        const int *__restrict__ skip, int64_t sks)
{
    __shared__ double2 sZ[TB][TB + 1];
    __shared__ double2 sXI[TB][32];
    __shared__ double2 sXJ[TB][32];
    __shared__ int32_t live[32];
    const int64_t b = blockIdx.x;
    const int32_t p = items[3 * b], u = items[3 * b + 1], g = items[3 * b + 2];
    const GProb P = probs[p];
    const int32_t I = __builtin_amdgcn_readfirstlane(P.units[3 * u]);
    const int32_t J0 = __builtin_amdgcn_readfirstlane(P.units[3 * u + 1]);
    const int32_t J1 = __builtin_amdgcn_readfirstlane(P.units[3 * u + 2]);
    const int32_t uo = __builtin_amdgcn_readfirstlane(u - P.unit_ptr[I]);
    const int32_t cb = P.c0 + g * G, ce = min(min(P.c1, cb + G), cb + 32);
    const int nc = ce - cb;
    const int t = threadIdx.x, lane = t & 63, w = t >> 6, ni = lane & 15, nk = lane >> 4;
    if (t < 32) live[t] = (t < nc && !(skip && skip[int64_t(cb + t) * sks])) ? 1 : 0;
    __syncthreads();
    int hi = 0;
    for (int c = 0; c < nc; ++c)
        if (live[c]) hi = c + 1;
    if (hi == 0) return;   // uniform over the block
    const int halves = hi <= 16 ? 1 : 2;
    const double2 *Z = static_cast<const double2 *>(P.Z);
    const double2 *Xc = reinterpret_cast<const double2 *>(X);
    // staging as in the FP32 pass: column t & 31 of the vectors (rows t/32 + 8 i),
    // entries t + 256 i of the tile
    const int sc = t & 31, sr = t >> 5;
    const bool slive = live[sc] != 0;
    const int64_t sxo = slive ? gc.xoff[cb + sc] + gc.xstep * P.N : 0;
    auto load_x = [&](double2 (&xv)[8], int32_t blk) {
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int64_t row = int64_t(blk) * TB + sr + 8 * q;
            xv[q] = (slive && row < P.N) ? gload_d2(Xc, sxo + row) : make_double2(0.0, 0.0);
        }
    };
    auto put_x = [&](double2 (*dst)[32], const double2 (&xv)[8]) {
#pragma unroll
        for (int q = 0; q < 8; ++q) dst[sr + 8 * q][sc] = xv[q];
    };
    auto load_z = [&](double2 (&zv)[16], int32_t J) {
        const double2 *tile = Z + tile_of(I, J, P.nT) * TB * TB + t;
#pragma unroll
        for (int q = 0; q < 16; ++q) zv[q] = gload_d2(tile, 256 * q);
    };
    auto put_z = [&](const double2 (&zv)[16]) {
#pragma unroll
        for (int q = 0; q < 16; ++q) sZ[(t >> 6) + 4 * q][t & 63] = zv[q];
    };
    auto chain = [&](f64x4g (&ar)[2], f64x4g (&ai)[2], bool transposed, double2 (*xs)[32]) {
        for (int k0 = 0; k0 < TB; k0 += 4) {
            const double2 z = transposed ? sZ[k0 + nk][16 * w + ni] : sZ[16 * w + ni][k0 + nk];
#pragma unroll
            for (int c = 0; c < 2; ++c) {
                if (c >= halves) break;
                const double2 x = xs[k0 + nk][16 * c + ni];
                ar[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(z.x, x.x, ar[c], 0, 0, 0);
                ar[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(-z.y, x.y, ar[c], 0, 0, 0);
                ai[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(z.x, x.y, ai[c], 0, 0, 0);
                ai[c] = __builtin_amdgcn_mfma_f64_16x16x4f64(z.y, x.x, ai[c], 0, 0, 0);
            }
        }
    };
    auto store = [&](const f64x4g (&ar)[2], const f64x4g (&ai)[2], int64_t slot) {
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            if (c >= halves) break;
            const int col = 16 * c + ni;
            if (!live[col]) continue;
            double *pv = part + (gc.poff[cb + col] * TB + slot * TB) * 2;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int r = 16 * w + nk + 4 * q;
                pv[2 * r] = ar[c][q];
                pv[2 * r + 1] = ai[c][q];
            }
        }
    };
    double2 xv[8];
    double2 zv[16];
    load_x(xv, I);
    put_x(sXI, xv);
    load_z(zv, J0);
    load_x(xv, J0);
    f64x4g rr[2], ri[2];
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int q = 0; q < 4; ++q) rr[c][q] = ri[c][q] = 0.0;
    for (int32_t J = J0; J < J1; ++J) {
        __syncthreads();   // the previous tile's LDS reads are done
        put_z(zv);
        put_x(sXJ, xv);
        __syncthreads();
        if (J + 1 < J1) {   // the next tile's loads go out before this tile's products
            load_z(zv, J + 1);
            load_x(xv, J + 1);
        }
        chain(rr, ri, false, sXJ);
        if (J != I) {
            f64x4g cr[2], ci[2];
#pragma unroll
            for (int c = 0; c < 2; ++c)
#pragma unroll
                for (int q = 0; q < 4; ++q) cr[c][q] = ci[c][q] = 0.0;
            chain(cr, ci, true, sXI);
            store(cr, ci, gload_i64(P.seg, J) + I);
        }
    }
    store(rr, ri, gload_i64(P.seg, I) + I + uo);
}

// y_I = sum of the partial vectors of row block I (column sums of tiles
// (J < I, I), then row sums of the units of tile row I), stored contiguously.
// Eight waves split the vectors (every eighth one) and their sums are added in
// wave order (deterministic).
template <typename T, bool SUB>
__device__ inline void reduce_rows(int64_t N, const int64_t *__restrict__ seg, int64_t I,
                                   const typename Cx<T>::type *__restrict__ pv, typename Cx<T>::type *__restrict__ y,
                                   const typename Cx<T>::type *__restrict__ b)
{
    using V2 = typename Cx<T>::type;
    const int r = threadIdx.x & 63, w = threadIdx.x >> 6;
    pv += seg[I] * TB;
    const int64_t K = seg[I + 1] - seg[I];
    V2 a = { 0, 0 };
#pragma unroll 4
    for (int64_t q = w; q < K; q += 8) a += pv[q * TB + r];
    __shared__ V2 red[8][TB];
    red[w][r] = a;
    __syncthreads();
    if (w != 0) return;
    a = red[0][r];
#pragma unroll
    for (int q = 1; q < 8; ++q) a += red[q][r];
    const int64_t m = I * TB + r;
    if (m < N) {
        if (SUB) y[m] = b[m] - a;
        else y[m] = a;
    }
}

// The same with FP32 partial sums (the matrix-core pass stores its FP32
// accumulators as they are), added in FP64.
template <bool SUB>
__device__ inline void reduce_rows_f(int64_t N, const int64_t *__restrict__ seg, int64_t I,
                                     const float2 *__restrict__ pv, double2 *__restrict__ y,
                                     const double2 *__restrict__ b)
{
    const int r = threadIdx.x & 63, w = threadIdx.x >> 6;
    pv += seg[I] * TB;
    const int64_t K = seg[I + 1] - seg[I];
    double2 a = { 0, 0 };
#pragma unroll 4
    for (int64_t q = w; q < K; q += 8) {
        const float2 v = pv[q * TB + r];
        a.x += double(v.x);
        a.y += double(v.y);
    }
    __shared__ double2 red[8][TB];
    red[w][r] = a;
    __syncthreads();
    if (w != 0) return;
    a = red[0][r];
#pragma unroll
    for (int q = 1; q < 8; ++q) a += red[q][r];
    const int64_t m = I * TB + r;
    if (m < N) {
        if (SUB) y[m] = b[m] - a;
        else y[m] = a;
    }
}

template <typename T, bool SUB>
__global__ __launch_bounds__(512) void k_sym_reduce(int64_t N, const int64_t *__restrict__ seg, int64_t nslots,
                                                    const T *__restrict__ part, T *__restrict__ Y, int64_t ldy,
                                                    const T *__restrict__ B, int64_t ldb,
                                                    const int *__restrict__ skip, int64_t sks)
{
    using V2 = typename Cx<T>::type;
    const int64_t I = blockIdx.x, v = blockIdx.y;
    if (skip && skip[v * sks]) return;
    reduce_rows<T, SUB>(N, seg, I, reinterpret_cast<const V2 *>(part) + v * nslots * TB,
                        reinterpret_cast<V2 *>(Y) + v * ldy, SUB ? reinterpret_cast<const V2 *>(B) + v * ldb : nullptr);
}

// Grouped reduce: block b is the item (column c, row block I).
template <typename T, bool SUB>
__global__ __launch_bounds__(512) void k_sym_reduce_g(const GProb *__restrict__ probs, GCols gc,
                                                      const int32_t *__restrict__ items, const T *__restrict__ part,
                                                      T *__restrict__ Y, const T *__restrict__ B,
                                                      const int *__restrict__ skip, int64_t sks)
{
    using V2 = typename Cx<T>::type;
    const int64_t b = blockIdx.x;
    const int32_t c = items[2 * b], I = items[2 * b + 1];
    if (skip && skip[int64_t(c) * sks]) return;
    const GProb P = probs[gc.prob[c]];
    reduce_rows<T, SUB>(P.N, P.seg, I, reinterpret_cast<const V2 *>(part) + gc.poff[c] * TB,
                        reinterpret_cast<V2 *>(Y) + gc.yoff[c],
                        SUB ? reinterpret_cast<const V2 *>(B) + gc.yoff[c] : nullptr);
}

// Grouped reduce of the matrix-core pass's FP32 partial sums (FP64 sums, FP64 vectors)
template <bool SUB>
__global__ __launch_bounds__(512) void k_sym_reduce_gf(const GProb *__restrict__ probs, GCols gc,
                                                       const int32_t *__restrict__ items, const float *__restrict__ part,
                                                       double *__restrict__ Y, const double *__restrict__ B,
                                                       const int *__restrict__ skip, int64_t sks)
{
    const int64_t b = blockIdx.x;
    const int32_t c = items[2 * b], I = items[2 * b + 1];
    if (skip && skip[int64_t(c) * sks]) return;
    const GProb P = probs[gc.prob[c]];
    reduce_rows_f<SUB>(P.N, P.seg, I, reinterpret_cast<const float2 *>(part) + gc.poff[c] * TB,
                       reinterpret_cast<double2 *>(Y) + gc.yoff[c], SUB ? reinterpret_cast<const double2 *>(B) + gc.yoff[c] : nullptr);
}

// The full matrix from the packed tiles: a block reads RPB rows of a tile once, writes
// them as they lie and, through LDS, their columns as rows of the mirrored block, in runs
// of 64 and RPB entries (one thread per output entry read the mirrored half 1 KiB apart, lane by
// lane: 7680 unknowns 444 -> 277 us, 5.1 TB/s).  RPB: the whole tile, or a quarter where
// there are fewer tiles than CUs.
template <typename T, typename O, int RPB>
__global__ __launch_bounds__(256) void k_unpack(const T *__restrict__ Zp, int64_t N, int64_t nT,
                                                typename Cx<O>::type *__restrict__ out)
{
    using V2 = typename Cx<T>::type;
    using W2 = typename Cx<O>::type;
    __shared__ V2 sz[RPB][TB + 1];
    int64_t I, J;
    tile_decode(blockIdx.x, nT, I, J);
    const int r0 = RPB == TB ? 0 : int(blockIdx.y) * RPB;
    const V2 *Z = reinterpret_cast<const V2 *>(Zp) + int64_t(blockIdx.x) * TB * TB + r0 * TB;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int64_t m0 = I * TB + r0, n0 = J * TB;
#pragma unroll
    for (int i = 0; i < RPB / 4; ++i) {
        const int r = w + 4 * i;
        const V2 z = __builtin_nontemporal_load(Z + r * TB + lane);
        sz[r][lane] = z;
        if (m0 + r < N && n0 + lane < N) __builtin_nontemporal_store(W2{ O(z.x), O(z.y) }, out + (m0 + r) * N + n0 + lane);
    }
    if (I == J) return;
    __syncthreads();
#pragma unroll
    for (int i = 0; i < RPB / 4; ++i) {
        const int r = RPB == TB ? lane : threadIdx.x % RPB, c = RPB == TB ? w + 4 * i : (threadIdx.x + 256 * i) / RPB;
        const V2 z = sz[r][c];
        if (n0 + c < N && m0 + r < N) __builtin_nontemporal_store(W2{ O(z.x), O(z.y) }, out + (n0 + c) * N + m0 + r);
    }
}

// One wave per sampled row i: (T x)_i from the packed tiles (row i of tiles
// (I, J >= I), column i of tiles (J < I, I)), then |b_i - (T x)_i|^2.
__global__ __launch_bounds__(256) void k_sampled_rows(const double2 *__restrict__ Zp, int64_t N, int64_t nT,
                                                      int64_t S, const int64_t *__restrict__ rows,
                                                      const double2 *__restrict__ B, const double2 *__restrict__ X,
                                                      double *__restrict__ out, const int *__restrict__ mask)
{
    const int64_t v = blockIdx.y;
    if (!mask[v]) return;
    const int lane = threadIdx.x & 63;
    const int64_t s = int64_t(blockIdx.x) * 4 + (threadIdx.x >> 6);
    if (s >= S) return;
    const int64_t i = rows[v * S + s];
    const int64_t I = i / TB, rr = i % TB;
    const double2 *x = X + v * N;
    double ar = 0.0, ai = 0.0;
    for (int64_t J = 0; J < nT; ++J) {
        const int64_t n = J * TB + lane;
        if (n >= N) continue;
        const double2 z = J >= I ? Zp[tile_of(I, J, nT) * TB * TB + rr * TB + lane]
                                 : Zp[tile_of(J, I, nT) * TB * TB + lane * TB + rr];
        const double2 xv = x[n];
        ar += z.x * xv.x - z.y * xv.y;
        ai += z.x * xv.y + z.y * xv.x;
    }
    ar = wsum(ar);
    ai = wsum(ai);
    if (lane == 0) {
        const double2 b = B[v * N + i];
        const double dr = b.x - ar, di = b.y - ai;
        out[v * S + s] = dr * dr + di * di;
    }
}

__global__ void k_convert_d2f(const double *__restrict__ a, float *__restrict__ b, int64_t n)
{
    for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += int64_t(gridDim.x) * blockDim.x)
        b[i] = float(a[i]);
}
__global__ void k_convert_f2d(const float *__restrict__ a, double *__restrict__ b, int64_t n)
{
    for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += int64_t(gridDim.x) * blockDim.x)
        b[i] = double(a[i]);
}
__global__ void k_nonfinite(const double *__restrict__ a, int64_t n, int *__restrict__ flag)
{
    for (int64_t i = int64_t(blockIdx.x) * blockDim.x + threadIdx.x; i < n; i += int64_t(gridDim.x) * blockDim.x)
        if (!isfinite(a[i])) *flag = 1;
}

// Tile-pass variant: register double buffering of the next tile (default) or
// not; BIE_SYM_PREFETCH=0 selects the plain form (kept for measurement).
int sym_prefetch()
{
    static int v = [] {
        const char *e = getenv("BIE_SYM_PREFETCH");
        return e ? atoi(e) : 1;
    }();
    return v;
}

// Star-split product (Sec. VI-A): T x = T_A' x + Sigma V' Sigma^T x.
// u = Sigma^T x: u_p = sum over the three edges m of triangle p of s x_m.
template <typename T>
__global__ __launch_bounds__(256) void k_star_gather(int64_t F, const int32_t *__restrict__ slot_m,
                                                     const int8_t *__restrict__ sgn, const T *__restrict__ X,
                                                     int64_t ldx, T *__restrict__ U, const int *__restrict__ skip,
                                                     int64_t sks)
{
    using V2 = typename Cx<T>::type;
    const int64_t v = blockIdx.y;
    if (skip && skip[v * sks]) return;
    const V2 *x = reinterpret_cast<const V2 *>(X) + v * ldx;
    V2 *u = reinterpret_cast<V2 *>(U) + v * F;
    for (int64_t p = int64_t(blockIdx.x) * 256 + threadIdx.x; p < F; p += int64_t(gridDim.x) * 256) {
        V2 a = { 0, 0 };
#pragma unroll
        for (int e = 0; e < 3; ++e) {
            const V2 xm = x[slot_m[3 * p + e]];
            if (sgn[3 * p + e] > 0) a += xm;
            else a -= xm;
        }
        u[p] = a;
    }
}

// y_m += w_{c+(m)} - w_{c-(m)} (SUB: -=), w = V' u
template <typename T, bool SUB>
__global__ __launch_bounds__(256) void k_star_scatter(int64_t N, int64_t F, const int4 *__restrict__ rwg4,
                                                      const T *__restrict__ W, T *__restrict__ Y, int64_t ldy,
                                                      const int *__restrict__ skip, int64_t sks)
{
    using V2 = typename Cx<T>::type;
    const int64_t v = blockIdx.y;
    if (skip && skip[v * sks]) return;
    const V2 *w = reinterpret_cast<const V2 *>(W) + v * F;
    V2 *y = reinterpret_cast<V2 *>(Y) + v * ldy;
    for (int64_t m = int64_t(blockIdx.x) * 256 + threadIdx.x; m < N; m += int64_t(gridDim.x) * 256) {
        const int4 e = rwg4[m];
        const V2 d = w[e.x] - w[e.y];
        if (SUB) y[m] -= d;
        else y[m] += d;
    }
}

template <typename M, typename T, bool CONJ, bool SUB>
void launch_product(const Packed &pk, void *part, const void *Z, const void *X, int64_t ldx, void *Y, int64_t ldy,
                    const void *B, int64_t ldb, int64_t R, const int *skip, int64_t sks, hipStream_t s,
                    bool profile = true)
{
    const dim3 grid(unsigned(pk.nruns), unsigned(R));
    if (profile) prof::begin(0, s, R);
    // non-temporal tile loads for the FP64 matrix, cached loads for the FP32
    // one (measured: 92 vs 144 us, 52 vs 47 us at N = 7680)
    constexpr bool NT = sizeof(M) == 8;
    // Several vectors share the tile reads in groups of up to 3 (FP64 vectors; 4
    // spill) or 4, as even as they come.  A matrix below 10 MB comes from the L2s whatever
    // reads it, and one block per vector fills more CUs (us, a block per vector / groups, of
    // 3 and 16 vectors: FP64, 882 unknowns, 6.9 MB 9 / 10, 15 / 17; 1152, 11.2 MB 12 / 10,
    // 29 / 23; FP32, 1458, 9.0 MB 9 / 9, 18 / 22; 2178, 20.6 MB 16 / 12, 54 / 33).  With many
    // vectors every CU is busy either way, and FP64 tiles are better read once (648
    // unknowns, 64 and 256 vectors 30 / 29, 123 / 99; 882 45 / 37, 181 / 134).
    constexpr int MAXNC = sizeof(T) == 8 ? 3 : 4;
    auto several = [&](auto kern, int nc) {
        const int64_t G = (R + nc - 1) / nc;
        hipLaunchKernelGGL(kern, dim3(unsigned((pk.nruns + 7) / 8 * 8 * G)), dim3(512), 0, s, int(pk.nruns), (const M *)Z,
                           pk.N, pk.nT, pk.units, pk.unit_ptr, pk.run_ptr, pk.seg, pk.nslots, int(G), R, (const T *)X, ldx,
                           (T *)part, skip, sks);
    };
    if (R > 1 && (pk.ntiles * TB * TB * int64_t(2 * sizeof(M)) >= 10000000 || (sizeof(M) == 8 && pk.ntiles * R >= 5000))) {
        const int64_t G = (R + MAXNC - 1) / MAXNC, nc = (R + G - 1) / G;
        // a matrix beyond the 256 MB last-level cache is streamed past it (us, cached /
        // streamed, 2, 3 and 6 FP64 vectors: 5202 unknowns, 213 MiB 44 / 53, 50 / 62, 82 / 94;
        // 7200, 403 MiB 109 / 99, 120 / 113, 162 / 160)
        const bool stream = pk.ntiles * TB * TB * int64_t(2 * sizeof(M)) > (int64_t(256) << 20);
        if (nc == 2) stream ? several(k_sym_tiles_n<M, T, CONJ, 2, true>, 2) : several(k_sym_tiles_n<M, T, CONJ, 2, false>, 2);
        else if (nc == 3) stream ? several(k_sym_tiles_n<M, T, CONJ, 3, true>, 3) : several(k_sym_tiles_n<M, T, CONJ, 3, false>, 3);
        else if constexpr (MAXNC == 4)
            stream ? several(k_sym_tiles_n<M, T, CONJ, 4, true>, 4) : several(k_sym_tiles_n<M, T, CONJ, 4, false>, 4);
    } else if (sym_prefetch())
        hipLaunchKernelGGL((k_sym_tiles<M, T, CONJ, true, NT>), grid, dim3(256), 0, s, (const M *)Z, pk.N, pk.nT,
                           pk.units, pk.unit_ptr, pk.run_ptr, pk.seg, pk.nslots, (const T *)X, ldx, (T *)part,
                           skip, sks);
    else
        hipLaunchKernelGGL((k_sym_tiles<M, T, CONJ, false, NT>), grid, dim3(256), 0, s, (const M *)Z, pk.N, pk.nT,
                           pk.units, pk.unit_ptr, pk.run_ptr, pk.seg, pk.nslots, (const T *)X, ldx, (T *)part,
                           skip, sks);
    if (profile) prof::end(0, s);
    if (!Y) {   // the caller adds the partial sums
        BIE_HIP(hipGetLastError());
        return;
    }
    if (profile) prof::begin(3, s, R);
    hipLaunchKernelGGL((k_sym_reduce<T, SUB>), dim3(unsigned(pk.nT), unsigned(R)), dim3(512), 0, s, pk.N, pk.seg,
                       pk.nslots, (const T *)part, (T *)Y, ldy, (const T *)B, ldb, skip, sks);
    BIE_HIP(hipGetLastError());
    if (profile) prof::end(3, s);
}

}  // namespace

// Row pointers and partial-slot segments of a unit table sorted by tile row:
// row block I owns the column sums of tiles (J < I, I), then one row-sum slot
// per unit of tile row I.
static void unit_rows(int64_t nT, const std::vector<int32_t> &units, std::vector<int32_t> &uptr,
                      std::vector<int64_t> &seg)
{
    const int64_t nu = int64_t(units.size() / 3);
    uptr.assign(nT + 1, int32_t(nu));
    for (int64_t u = nu - 1; u >= 0; --u) uptr[units[3 * u]] = int32_t(u);
    for (int64_t I = nT - 1; I >= 0; --I) uptr[I] = std::min(uptr[I], uptr[I + 1]);
    seg.assign(nT + 1, 0);
    for (int64_t I = 0; I < nT; ++I) seg[I + 1] = seg[I] + I + (uptr[I + 1] - uptr[I]);
}

void build_units(int64_t nT, int U, std::vector<int32_t> &units, std::vector<int32_t> &uptr,
                 std::vector<int64_t> &seg)
{
    units.clear();
    for (int64_t I = 0; I < nT; ++I)
        for (int64_t J0 = I; J0 < nT; J0 += U) {
            units.push_back(int32_t(I));
            units.push_back(int32_t(J0));
            units.push_back(int32_t(std::min<int64_t>(nT, J0 + U)));
        }
    unit_rows(nT, units, uptr, seg);
}

// Balanced runs: the T = nT (nT + 1) / 2 stored tiles in row-major order
// (I, J >= I) are cut into nb runs [T b / nb, T (b+1) / nb) of equal length
// to within one tile, and each run into units at the ends of tile rows; run b
// is units rptr[b] .. rptr[b+1]-1.  With nb = 512 (two 4-wave blocks on each of
// the 256 CUs) every block of a single-vector product has the same work and
// all are resident at once; small matrices take fewer runs (at least 8 tiles
// each: a run's fixed cost is loading x and writing its row sums).  Selected
// with BIE_SYM_UNIT=0.
void build_runs(int64_t nT, int64_t nb, std::vector<int32_t> &units, std::vector<int32_t> &uptr,
                std::vector<int64_t> &seg, std::vector<int32_t> &rptr)
{
    const int64_t T = nT * (nT + 1) / 2;
    nb = std::max<int64_t>(1, std::min(nb, T));
    units.clear();
    rptr.assign(nb + 1, 0);
    int64_t I = 0, J = 0, t = 0;
    for (int64_t b = 0; b < nb; ++b) {
        rptr[b] = int32_t(units.size() / 3);
        const int64_t t1 = T * (b + 1) / nb;
        while (t < t1) {
            const int64_t take = std::min(nT - J, t1 - t);
            units.push_back(int32_t(I));
            units.push_back(int32_t(J));
            units.push_back(int32_t(J + take));
            t += take;
            J += take;
            if (J == nT) J = ++I;
        }
    }
    rptr[nb] = int32_t(units.size() / 3);
    unit_rows(nT, units, uptr, seg);
}

// Tables of the packed n x n tiles with units of U tiles (U >= 1) or balanced
// runs (U = 0).
static void packed_setup_units(Packed &pk, int64_t n, int U)
{
    pk.N = n;
    pk.nT = (pk.N + TB - 1) / TB;
    pk.ntiles = pk.nT * (pk.nT + 1) / 2;
    pk.unit_len = U;
    std::vector<int32_t> units, uptr, rptr;
    std::vector<int64_t> seg;
    if (U > 0) {
        build_units(pk.nT, U, units, uptr, seg);
        rptr.resize(units.size() / 3 + 1);
        for (size_t b = 0; b < rptr.size(); ++b) rptr[b] = int32_t(b);
    } else {   // 512 runs, or fewer for small matrices: at least 8 tiles per run
        build_runs(pk.nT, std::max<int64_t>(1, std::min<int64_t>(512, pk.ntiles / 8)), units, uptr, seg, rptr);
    }
    pk.nunits = int64_t(units.size() / 3);
    pk.nruns = int64_t(rptr.size()) - 1;
    pk.nslots = seg[pk.nT];
    // seg, units, unit_ptr and run_ptr side by side, copied at once
    std::vector<char> image(seg.size() * sizeof(int64_t) + (units.size() + uptr.size() + rptr.size()) * sizeof(int32_t));
    size_t bytes = 0;
    auto put = [&](const auto &v) {
        const size_t at = bytes, n = v.size() * sizeof(v[0]);
        std::memcpy(image.data() + at, v.data(), n);
        bytes += n;
        return at;
    };
    const size_t o_seg = put(seg), o_units = put(units), o_uptr = put(uptr), o_rptr = put(rptr);
    char *d = nullptr;
    BIE_HIP(device_malloc(&d, bytes));
    pk.seg = reinterpret_cast<int64_t *>(d + o_seg);
    pk.units = reinterpret_cast<int32_t *>(d + o_units);
    pk.unit_ptr = reinterpret_cast<int32_t *>(d + o_uptr);
    pk.run_ptr = reinterpret_cast<int32_t *>(d + o_rptr);
    BIE_HIP(hipMemcpy(d, image.data(), bytes, hipMemcpyHostToDevice));
    pk.h_units = std::move(units);
    pk.h_unit_ptr = std::move(uptr);
    pk.h_seg = std::move(seg);
}

void packed_setup(Packed &pk, int64_t n, bool mat64) { packed_setup_units(pk, n, unit_tiles((n + TB - 1) / TB, mat64)); }

static std::string tune_key(int64_t N, bool mat64) { return "sym:" + std::to_string(N) + (mat64 ? ":f64" : ":f32"); }
static bool tuned_unit(const std::string &key, int &unit)
{
    std::vector<int> v;
    if (!tune_get(key, v) || v.size() != 1 || v[0] < 0 || v[0] > 64) return false;
    unit = v[0];
    return true;
}

// With the autotuner's units where it has met the size (tune_packed then has nothing to rebuild).
void packed_setup_tuned(Packed &pk, int64_t n, bool mat64)
{
    int unit = unit_tiles((n + TB - 1) / TB, mat64);
    if (!getenv("BIE_SYM_UNIT") && tune_enabled()) (void)tuned_unit(tune_key(n, mat64), unit);
    packed_setup_units(pk, n, unit);
}

void packed_free(Packed &pk)
{
    if (pk.seg) (void)hipFree(pk.seg);   // and the tables behind it
    if (pk.part) (void)hipFree(pk.part);
    pk.seg = nullptr;
    pk.units = pk.unit_ptr = pk.run_ptr = nullptr;
    pk.part = nullptr;
    pk.part_R = 0;
}

// part: the partial sums, R x nslots x 64 complex T (the operator's buffer, or
// the static scratch of the allocation-free entry point, which also skips the
// profiling events)
template <typename M, typename T>
void dispatch(const Packed &pk, const void *Z, const void *X, int64_t ldx, void *Y, int64_t ldy, const void *B,
              int64_t ldb, int64_t R, const int *skip, int64_t sks, bool conj, hipStream_t s, void *part = nullptr)
{
    const bool profile = part == nullptr;
    if (!part) part = pk.part;
    if (B) launch_product<M, T, false, true>(pk, part, Z, X, ldx, Y, ldy, B, ldb, R, skip, sks, s, profile);
    else if (conj) launch_product<M, T, true, false>(pk, part, Z, X, ldx, Y, ldy, nullptr, 0, R, skip, sks, s, profile);
    else launch_product<M, T, false, false>(pk, part, Z, X, ldx, Y, ldy, nullptr, 0, R, skip, sks, s, profile);
}

// partial-sum buffer of a packed product for R vectors (sized for complex128)
static void ensure_part(Packed &pk, int64_t R, hipStream_t s)
{
    if (pk.part_R >= R) return;
    BIE_HIP(hipStreamSynchronize(s));
    if (pk.part) (void)hipFree(pk.part);
    pk.part = nullptr;
    pk.part_R = 0;
    BIE_HIP(device_malloc(&pk.part, size_t(R) * size_t(pk.nslots) * TB * 16));
    pk.part_R = R;
}

// The packed product's work units for this operator: the autotuner's choice
// for (N, matrix precision) among the rule's units and, where those are of 8
// tiles, 4, 16 and balanced runs, else twice the rule's, timed (tile pass and
// reduction of one vector) the first time the size occurs; the operator's
// tables are rebuilt if the choice is not the rule's.
// Fixed by BIE_SYM_UNIT (measurement) or with tuning off.
void tune_packed(bie_op *op, hipStream_t s)
{
    if (op->star || getenv("BIE_SYM_UNIT") || !tune_enabled() || stream_capturing(s)) return;
    const bool mat64 = op->Z64 != nullptr;
    const void *Z = mat64 ? op->Z64 : op->Z32;
    if (!Z) return;
    const int64_t N = op->mesh.N;
    const std::string key = tune_key(N, mat64);
    std::vector<int> v(1);
    if (!tuned_unit(key, v[0])) {
        void *x = nullptr, *y = nullptr;
        BIE_HIP(device_malloc(&x, size_t(N) * 16));
        try {
            BIE_HIP(device_malloc(&y, size_t(N) * 16));
            BIE_HIP(hipMemsetAsync(x, 0, size_t(N) * 16, s));
            float best = 0.f;
            const int def = unit_tiles((N + TB - 1) / TB, mat64);
            v = { def };
            // below the rule's 8 tiles a launch is some microseconds: more launches, and the
            // next longer units (shorter ones cost the products of several vectors more than
            // this one vector gains)
            const std::vector<int> cand = def >= 8 ? std::vector<int>{ def, 4, 0, 16 } : std::vector<int>{ def, 2 * def };
            for (int U : cand) {
                Packed c;
                try {
                    packed_setup_units(c, N, U);
                    ensure_part(c, 1, s);
                    const float ms = time_launches(s, def >= 8 ? 10 : 20, [&]() {
                        if (mat64)
                            launch_product<double, double, false, false>(c, c.part, Z, x, N, y, N, nullptr, 0, 1,
                                                                         nullptr, 1, s, false);
                        else
                            launch_product<float, double, false, false>(c, c.part, Z, x, N, y, N, nullptr, 0, 1,
                                                                        nullptr, 1, s, false);
                    });
                    if (best == 0.f || ms < 0.97f * best) {   // the rule's unless clearly slower
                        best = ms;
                        v = { U };
                    }
                } catch (...) {
                    packed_free(c);
                    throw;
                }
                packed_free(c);
            }
        } catch (...) {
            (void)hipFree(x);
            if (y) (void)hipFree(y);
            throw;
        }
        BIE_HIP(hipStreamSynchronize(s));
        (void)hipFree(x);
        (void)hipFree(y);
        tune_put(key, v);
    }
    if (v[0] != op->pk.unit_len) {
        BIE_HIP(hipStreamSynchronize(s));
        packed_free(op->pk);
        packed_setup_units(op->pk, N, v[0]);
    }
}

// T x (conj: conj(T) x; B: B - T x) for the star-split operator: u = Sigma^T x,
// w = V' u, y = T_A' x (or B - T_A' x), y += Sigma w (or -=).
template <typename M, typename T>
static void star_product(bie_op *op, const void *Za, const void *Vm, const void *X, int64_t ldx, void *Y,
                         int64_t ldy, const void *B, int64_t ldb, int64_t R, const int *skip, int64_t sks, bool conj,
                         hipStream_t s)
{
    const int64_t N = op->mesh.N, F = op->mesh.F;
    if (op->star_R < R) {
        BIE_HIP(hipStreamSynchronize(s));
        if (op->star_buf) (void)hipFree(op->star_buf);
        op->star_buf = nullptr;
        op->star_R = 0;
        BIE_HIP(device_malloc(&op->star_buf, 2 * size_t(R) * size_t(F) * 16));
        op->star_R = R;
    }
    T *U = static_cast<T *>(op->star_buf), *W = U + 2 * R * F;
    const unsigned gx = unsigned(std::min<int64_t>((std::max(N, F) + 255) / 256, 1024));
    hipLaunchKernelGGL(k_star_gather<T>, dim3(gx, unsigned(R)), dim3(256), 0, s, F, op->tri.slot_m, op->tri.sgn,
                       (const T *)X, ldx, U, skip, sks);
    dispatch<M, T>(op->pkv, Vm, U, F, W, F, nullptr, 0, R, skip, sks, conj, s);
    dispatch<M, T>(op->pk, Za, X, ldx, Y, ldy, B, ldb, R, skip, sks, conj, s);
    if (B) hipLaunchKernelGGL((k_star_scatter<T, true>), dim3(gx, unsigned(R)), dim3(256), 0, s, N, F,
                              (const int4 *)op->tri.edges, W, (T *)Y, ldy, skip, sks);
    else hipLaunchKernelGGL((k_star_scatter<T, false>), dim3(gx, unsigned(R)), dim3(256), 0, s, N, F,
                            (const int4 *)op->tri.edges, W, (T *)Y, ldy, skip, sks);
    BIE_HIP(hipGetLastError());
}

void product(const bie_op *opc, int mat, bool vec64, const void *X, int64_t ldx, void *Y, int64_t ldy,
             const void *B, int64_t ldb, int64_t R, const int *skip, int64_t sks, bool conj, hipStream_t s)
{
    bie_op *op = const_cast<bie_op *>(opc);
    if (op->fast) {   // near entries + multilevel far field; every vector computed (no skip)
        if (!vec64 || conj) throw Error(BIE_EINVAL, "the fast operator takes complex128 vectors, no conjugate");
        fast_product(op, X, ldx, Y, ldy, B, ldb, R, s);
        return;
    }
    if (mat == MATBF16) {
        if (!op->Abf) throw Error(BIE_EINVAL, "no split-BF16 matrix stored");
        if (!vec64 || conj) throw Error(BIE_EINVAL, "the block product takes complex128 vectors, no conjugate");
        gemm_product(op, X, ldx, VEC_C128, Y, ldy, B, ldb, R, nullptr, s);
        return;
    }
    const bool mat64 = mat == MAT64;
    const void *Z = mat64 ? op->Z64 : op->Z32;
    if (!Z) throw Error(BIE_EINVAL, "matrix not stored in the requested precision");
    if (mat64 && !vec64) throw Error(BIE_EINVAL, "complex64 vectors need the FP32 matrix");
    ensure_part(op->pk, R, s);
    if (op->star) {
        const void *Vm = mat64 ? op->V64 : op->V32;
        ensure_part(op->pkv, R, s);
        if (mat64) star_product<double, double>(op, Z, Vm, X, ldx, Y, ldy, B, ldb, R, skip, sks, conj, s);
        else if (vec64) star_product<float, double>(op, Z, Vm, X, ldx, Y, ldy, B, ldb, R, skip, sks, conj, s);
        else star_product<float, float>(op, Z, Vm, X, ldx, Y, ldy, B, ldb, R, skip, sks, conj, s);
        return;
    }
    if (mat64) dispatch<double, double>(op->pk, Z, X, ldx, Y, ldy, B, ldb, R, skip, sks, conj, s);
    else if (vec64) dispatch<float, double>(op->pk, Z, X, ldx, Y, ldy, B, ldb, R, skip, sks, conj, s);
    else dispatch<float, float>(op->pk, Z, X, ldx, Y, ldy, B, ldb, R, skip, sks, conj, s);
}

// ----------------------------------------------------------------------------- allocation-free product
// For callers that cannot allocate (graph capture, serving loops): the
// partial sums live in this static array instead of the operator's buffer.
// Each device holds its own copy for the life of the process; host code
// reaches it only through the address hipGetSymbolAddress returns on that
// device (kept in scratch_dev), never through the array's name.
constexpr size_t NOALLOC_SCRATCH_BYTES = size_t(128) << 20;
static __device__ __align__(256) unsigned char scratch[NOALLOC_SCRATCH_BYTES];

namespace {
constexpr int MAX_DEVICES = 64;
std::mutex scratch_mu;
void *scratch_dev[MAX_DEVICES] = { nullptr };

// device address of the current device's scratch, looked up once per device
void *noalloc_scratch(int dev)
{
    if (dev < 0 || dev >= MAX_DEVICES) throw Error(BIE_EDEVICE, "device index beyond the scratch table");
    std::lock_guard<std::mutex> g(scratch_mu);
    if (!scratch_dev[dev]) {
        void *p = nullptr;
        BIE_HIP(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p) throw Error(BIE_EDEVICE, "hipGetSymbolAddress returned no address for the scratch array");
        scratch_dev[dev] = p;
    }
    return scratch_dev[dev];
}
}  // namespace

void product_noalloc(const bie_op *op, bool vec64, const void *X, void *Y, int64_t R, bool conj, hipStream_t s)
{
    if (op->star) throw Error(BIE_EINVAL, "the allocation-free product takes an assembled operator");
    const Packed &pk = op->pk;
    // Short units take up to twice the partial slots of long ones: a call is judged by units of 16
    // tiles, whatever the operator's are, and where its own do not fit made in several passes,
    // each of one vector at least: units too short for a large matrix are refused.
    int64_t most = pk.nT * (pk.nT - 1) / 2;
    for (int64_t I = 0; I < pk.nT; ++I) most += (pk.nT - I + 15) / 16;
    const int64_t slots = std::min(pk.nslots, most);
    const size_t per = TB * (vec64 ? 16 : 8), one = size_t(pk.nslots) * per,
                 need = std::max(size_t(R) * size_t(slots) * per, one);
    if (need > NOALLOC_SCRATCH_BYTES)
        throw Error(BIE_EINVAL, "partial sums of " + std::to_string(need) + " bytes exceed the " +
                                    std::to_string(NOALLOC_SCRATCH_BYTES) + "-byte scratch of the allocation-free "
                                    "product: use fewer vectors per call");
    int dev = -1;
    BIE_HIP(hipGetDevice(&dev));
    if (dev != op->device) throw Error(BIE_EINVAL, "the operator's device must be current");
    if (vec64 ? !op->Z64 && !op->Z32 : !op->Z32)
        throw Error(BIE_EINVAL, vec64 ? "no packed matrix stored" : "complex64 vectors need the FP32 matrix");
    void *part = noalloc_scratch(dev);
    const int64_t pass = int64_t(NOALLOC_SCRATCH_BYTES / one);
    const size_t vec = size_t(pk.N) * (vec64 ? 16 : 8);
    for (int64_t r0 = 0; r0 < R; r0 += pass) {
        const int64_t n = std::min(pass, R - r0);
        const void *x = static_cast<const char *>(X) + size_t(r0) * vec;
        void *y = static_cast<char *>(Y) + size_t(r0) * vec;
        if (!vec64) dispatch<float, float>(pk, op->Z32, x, pk.N, y, pk.N, nullptr, 0, n, nullptr, 1, conj, s, part);
        else if (op->Z64) dispatch<double, double>(pk, op->Z64, x, pk.N, y, pk.N, nullptr, 0, n, nullptr, 1, conj, s, part);
        else dispatch<float, double>(pk, op->Z32, x, pk.N, y, pk.N, nullptr, 0, n, nullptr, 1, conj, s, part);
    }
}

void grouped_product(bool mat64, const GProb *probs, const GCols &gc, const int32_t *items, int64_t nitems, int G,
                     const int32_t *ritems, int64_t nritems, const void *X, void *part, void *Y, const void *B,
                     const int *skip, int64_t sks, hipStream_t s, bool mfma)
{
    if (nitems == 0) return;
    const bool pf = sym_prefetch() != 0;
    if (mfma) {
        if (G > 32) throw Error(BIE_EINVAL, "the matrix-core grouped pass takes at most 32 columns per item");
        if (mat64)
            hipLaunchKernelGGL(k_sym_tiles_gm64, dim3(unsigned(nitems)), dim3(256), 0, s, probs, gc, items, G,
                               (const double *)X, (double *)part, skip, sks);
        else {   // FP32 partial sums, reduced here
            hipLaunchKernelGGL(k_sym_tiles_gm, dim3(unsigned(nitems)), dim3(256), 0, s, probs, gc, items, G,
                               (const double *)X, (float *)part, skip, sks);
            if (B) hipLaunchKernelGGL(k_sym_reduce_gf<true>, dim3(unsigned(nritems)), dim3(512), 0, s, probs, gc, ritems,
                                      (const float *)part, (double *)Y, (const double *)B, skip, sks);
            else hipLaunchKernelGGL(k_sym_reduce_gf<false>, dim3(unsigned(nritems)), dim3(512), 0, s, probs, gc, ritems,
                                    (const float *)part, (double *)Y, nullptr, skip, sks);
            BIE_HIP(hipGetLastError());
            return;
        }
    } else if (mat64) {
        if (pf) hipLaunchKernelGGL((k_sym_tiles_g<double, double, true>), dim3(unsigned(nitems)), dim3(256), 0, s, probs,
                                   gc, items, G, (const double *)X, (double *)part, skip, sks);
        else hipLaunchKernelGGL((k_sym_tiles_g<double, double, false>), dim3(unsigned(nitems)), dim3(256), 0, s,
                                probs, gc, items, G, (const double *)X, (double *)part, skip, sks);
    } else {
        if (pf) hipLaunchKernelGGL((k_sym_tiles_g<float, double, true>), dim3(unsigned(nitems)), dim3(256), 0, s, probs,
                                   gc, items, G, (const double *)X, (double *)part, skip, sks);
        else hipLaunchKernelGGL((k_sym_tiles_g<float, double, false>), dim3(unsigned(nitems)), dim3(256), 0, s, probs,
                                gc, items, G, (const double *)X, (double *)part, skip, sks);
    }
    if (B) hipLaunchKernelGGL((k_sym_reduce_g<double, true>), dim3(unsigned(nritems)), dim3(512), 0, s, probs, gc,
                              ritems, (const double *)part, (double *)Y, (const double *)B, skip, sks);
    else hipLaunchKernelGGL((k_sym_reduce_g<double, false>), dim3(unsigned(nritems)), dim3(512), 0, s, probs, gc,
                            ritems, (const double *)part, (double *)Y, nullptr, skip, sks);
    BIE_HIP(hipGetLastError());
}

void unpack_full(const bie_op *op, bool from64, bool to64, void *dst, hipStream_t s)
{
    const Packed &pk = op->pk;
    auto go = [&](auto whole, auto quarter, const auto *Z, auto *out) {
        if (pk.ntiles < 256) hipLaunchKernelGGL(quarter, dim3(unsigned(pk.ntiles), 4), dim3(256), 0, s, Z, pk.N, pk.nT, out);
        else hipLaunchKernelGGL(whole, dim3(unsigned(pk.ntiles)), dim3(256), 0, s, Z, pk.N, pk.nT, out);
    };
    const double *Z64 = static_cast<const double *>(op->Z64);
    const float *Z32 = static_cast<const float *>(op->Z32);
    if (from64) go(k_unpack<double, double, TB>, k_unpack<double, double, TB / 4>, Z64, static_cast<nd2 *>(dst));
    else if (to64) go(k_unpack<float, double, TB>, k_unpack<float, double, TB / 4>, Z32, static_cast<nd2 *>(dst));
    else go(k_unpack<float, float, TB>, k_unpack<float, float, TB / 4>, Z32, static_cast<nf2 *>(dst));
    BIE_HIP(hipGetLastError());
}

void sampled_residual(const bie_op *op, const void *B, const void *X, int64_t R, int64_t S, const int64_t *rows,
                      double *out, const int *mask, hipStream_t s)
{
    if (!op->Z64) throw Error(BIE_EINVAL, "the random-sampling criterion needs the FP64 matrix");
    const Packed &pk = op->pk;
    hipLaunchKernelGGL(k_sampled_rows, dim3(unsigned((S + 3) / 4), unsigned(R)), dim3(256), 0, s,
                       (const double2 *)op->Z64, pk.N, pk.nT, S, rows, (const double2 *)B, (const double2 *)X, out,
                       mask);
    BIE_HIP(hipGetLastError());
}

void convert_c128_to_c64(const void *src, void *dst, int64_t n, hipStream_t s)
{
    hipLaunchKernelGGL(k_convert_d2f, dim3(2048), dim3(256), 0, s, (const double *)src, (float *)dst, 2 * n);
    BIE_HIP(hipGetLastError());
}

void convert_c64_to_c128(const void *src, void *dst, int64_t n, hipStream_t s)
{
    hipLaunchKernelGGL(k_convert_f2d, dim3(2048), dim3(256), 0, s, (const float *)src, (double *)dst, 2 * n);
    BIE_HIP(hipGetLastError());
}

bool has_nonfinite(const void *x, int64_t n_doubles, hipStream_t s)
{
    int *flag = nullptr;
    BIE_HIP(device_malloc(&flag, sizeof(int)));
    BIE_HIP(hipMemsetAsync(flag, 0, sizeof(int), s));
    hipLaunchKernelGGL(k_nonfinite, dim3(1024), dim3(256), 0, s, (const double *)x, n_doubles, flag);
    int h = 0;
    BIE_HIP(hipMemcpyAsync(&h, flag, sizeof(int), hipMemcpyDeviceToHost, s));
    BIE_HIP(hipStreamSynchronize(s));
    (void)hipFree(flag);
    return h != 0;
}

}  // namespace bie
