// Touching or near triangle pairs on the device.
//
// A pair (p <= q) is flagged if the triangles share a vertex or if
// |c_p - c_q|^2 < (near_factor max(longest_p, longest_q))^2, decided by the same
// FP64 operations in the same order as the host search of mesh.cpp (products and
// sums rounded one by one), so both give the same list.
//
// Every pair is tested: a block takes PR rows p in scalar registers and its 16
// waves walk their shares of the triangles q in runs of 64, so that a triangle q is
// read once for PR tests.  One launch counts, a scan places the rows, and a second
// launch counts each wave's share again and writes the partners in ascending
// order.  FP64 vector issue bounds it, at about 15 instructions per 64 pairs and
// row.  The host search is linear in the triangles but takes 0.6 to 0.9 us each
// (a hash grid, a sort per row): at 5292 triangles 4.7 ms against 0.27 with both
// launches, the upload and the waits.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cfloat>
#include <cmath>
#include <utility>
#include <vector>

#include "bie_internal.hpp"

namespace bie {

// The device search grows with the square of the triangles.  A fast operator, which
// alone has so many, needs the list in the mesh's order and in the device's: two searches
// here, on the host a search and a sort.  ms, device / host: 80 688 triangles 25 / 142,
// 326 700 300 / 590, 480 000 630 / 880, 691 200 1280 / 1280, 1 044 300 2870 / 1940.
bool near_on_device(int64_t F) { return F <= 655360; }

namespace {

constexpr int PR = 8;    // rows per block
constexpr int PW = 16;   // waves per block

struct Tri {   // one triangle of the search, read by its position
    double c[3], longest;
    int32_t v[3], pad;
};

template <bool WRITE>
__global__ __launch_bounds__(64 * PW) void k_near(int64_t F, const Tri *__restrict__ tri, double near_factor,
                                                  double slack, int64_t *__restrict__ ptr,
                                                  int32_t *__restrict__ list)
{
    __shared__ int32_t cnt[PW][PR];
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int64_t p0 = int64_t(blockIdx.x) * PR;
    const int64_t share = (F - p0 + 64 * PW - 1) / (64 * PW) * 64, qa = p0 + w * share, qb = min(F, qa + share);
    // f(r, q, hit) for every row r and triangle q of the wave's share
    auto sweep = [&](auto f) {
        for (int64_t q0 = qa; q0 < qb; q0 += 64) {
            const int64_t q = q0 + lane;
            const Tri b = tri[q < F ? q : F - 1];
#pragma unroll
            for (int r = 0; r < PR; ++r) {
#pragma clang fp contract(off)
                const int64_t p = p0 + r;
                if (p >= F) break;   // uniform
                const Tri &a = tri[p];
                const double d0 = a.c[0] - b.c[0], d1 = a.c[1] - b.c[1], d2 = a.c[2] - b.c[2];
                const double dd = d0 * d0 + d1 * d1 + d2 * d2;
                const double L = fmax(a.longest, b.longest);
                const double thr = near_factor * L;
                const bool in = q < qb && q >= p;
                bool hit = in && dd < thr * thr;
                // triangles that share a vertex lie within 4/3 of the longest edge, the rounding
                // of their centroids (slack) apart
                const double reach = 1.5 * L + slack;
                if (__any(in && !hit && dd < reach * reach)) {
                    bool touch = false;
#pragma unroll
                    for (int i = 0; i < 3; ++i)
#pragma unroll
                        for (int j = 0; j < 3; ++j) touch = touch || a.v[i] == b.v[j];
                    hit = hit || (in && touch);
                }
                f(r, q, hit);
            }
        }
    };
    int32_t n[PR] = {};
    sweep([&](int r, int64_t, bool hit) { n[r] += __popcll(__ballot(hit)); });
    if (lane == 0)
#pragma unroll
        for (int r = 0; r < PR; ++r) cnt[w][r] = n[r];
    __syncthreads();
    if (!WRITE) {
        if (threadIdx.x < PR && p0 + threadIdx.x < F) {
            int64_t s = 0;
            for (int v = 0; v < PW; ++v) s += cnt[v][threadIdx.x];
            ptr[p0 + threadIdx.x] = s;
        }
        return;
    }
    int64_t at[PR];
#pragma unroll
    for (int r = 0; r < PR; ++r) {
        at[r] = p0 + r < F ? ptr[p0 + r] : 0;
        for (int v = 0; v < w; ++v) at[r] += cnt[v][r];
    }
    sweep([&](int r, int64_t q, bool hit) {
        const uint64_t m = __ballot(hit);
        if (hit) list[at[r] + __popcll(m & ((uint64_t(1) << lane) - 1))] = int32_t(q);
        at[r] += __popcll(m);
    });
}

// exclusive scan of n counts in place; ptr[n] = their sum (one block)
__global__ __launch_bounds__(1024) void k_scan(int64_t n, int64_t *__restrict__ ptr)
{
    __shared__ int64_t part[1024];
    const int t = threadIdx.x;
    const int64_t ch = (n + 1023) / 1024, a = min(n, t * ch), b = min(n, a + ch);
    int64_t s = 0;
    for (int64_t i = a; i < b; ++i) s += ptr[i];
    part[t] = s;
    __syncthreads();
    for (int o = 1; o < 1024; o <<= 1) {
        const int64_t v = t >= o ? part[t - o] : 0;
        __syncthreads();
        part[t] += v;
        __syncthreads();
    }
    int64_t run = t ? part[t - 1] : 0;
    for (int64_t i = a; i < b; ++i) {
        const int64_t c = ptr[i];
        ptr[i] = run;
        run += c;
    }
    if (t == 1023) ptr[n] = part[1023];
}

// the pairs (p, partner) of a search, renamed by rank (null: as they are), lower first
__global__ __launch_bounds__(256) void k_pairs_of(int64_t F, const int64_t *__restrict__ ptr,
                                                  const int32_t *__restrict__ list, const int32_t *__restrict__ rank,
                                                  int32_t *__restrict__ pairs)
{
    const int64_t p = int64_t(blockIdx.x) * 4 + (threadIdx.x >> 6);
    if (p >= F) return;
    for (int64_t e = ptr[p] + (threadIdx.x & 63); e < ptr[p + 1]; e += 64) {
        const int32_t a = rank ? rank[p] : int32_t(p), b = rank ? rank[list[e]] : list[e];
        pairs[2 * e] = min(a, b);
        pairs[2 * e + 1] = max(a, b);
    }
}

int32_t *pairs_of(const NearDev &nd, int64_t F, const int32_t *rank, hipStream_t s)
{
    int32_t *out = nullptr;
    BIE_HIP(device_malloc(&out, std::max<int64_t>(nd.n, 1) * 2 * sizeof(int32_t)));
    hipLaunchKernelGGL(k_pairs_of, dim3(unsigned((F + 3) / 4)), dim3(256), 0, s, F, nd.ptr, nd.list, rank, out);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) (void)hipFree(out);
    BIE_HIP(e);
    return out;
}

// device memory that is freed with the scope
struct Temp {
    void *p = nullptr;
    explicit Temp(size_t bytes) { BIE_HIP(device_malloc(&p, std::max<size_t>(bytes, 1))); }
    ~Temp() { (void)hipFree(p); }
    Temp(const Temp &) = delete;
    Temp &operator=(const Temp &) = delete;
};

}  // namespace

void near_search(const Mesh &M, double near_factor, const std::vector<int32_t> *order, NearDev &out, hipStream_t s)
{
    const int64_t F = M.F;
    std::vector<Tri> h(F);
    for (int64_t r = 0; r < F; ++r) {
        const int64_t t = order ? (*order)[r] : r;
        for (int d = 0; d < 3; ++d) {
            h[r].c[d] = M.cent[3 * t + d];
            h[r].v[d] = M.T[3 * t + d];
        }
        h[r].longest = M.longest[t];
        h[r].pad = 0;
    }
    // a centroid is off by up to 4/3 eps of the largest coordinate on each axis
    double most = 0.0;
    for (double x : M.V) most = std::max(most, std::fabs(x));
    const double slack = 8.0 * DBL_EPSILON * most;
    Temp tri(size_t(F) * sizeof(Tri));
    BIE_HIP(hipMemcpyAsync(tri.p, h.data(), size_t(F) * sizeof(Tri), hipMemcpyHostToDevice, s));
    BIE_HIP(device_malloc(&out.ptr, size_t(F + 1) * sizeof(int64_t)));
    const dim3 grid(unsigned((F + PR - 1) / PR));
    hipLaunchKernelGGL(k_near<false>, grid, dim3(64 * PW), 0, s, F, (const Tri *)tri.p, near_factor, slack, out.ptr, nullptr);
    hipLaunchKernelGGL(k_scan, dim3(1), dim3(1024), 0, s, F, out.ptr);
    BIE_HIP(hipGetLastError());
    BIE_HIP(hipMemcpyAsync(&out.n, out.ptr + F, sizeof(int64_t), hipMemcpyDeviceToHost, s));
    BIE_HIP(hipStreamSynchronize(s));
    BIE_HIP(device_malloc(&out.list, std::max<int64_t>(out.n, 1) * sizeof(int32_t)));
    hipLaunchKernelGGL(k_near<true>, grid, dim3(64 * PW), 0, s, F, (const Tri *)tri.p, near_factor, slack, out.ptr, out.list);
    BIE_HIP(hipGetLastError());
    BIE_HIP(hipStreamSynchronize(s));   // the triangles' copy ends with the call
}

void flag_pairs(bie_op *op, double near_factor, bool device_list, hipStream_t s)
{
    Mesh &M = op->mesh;
    if (near_on_device(M.F)) {
        const std::vector<int32_t> &rank = op->tri.rank;
        NearDev nd;
        near_search(M, near_factor, nullptr, nd, s);
        std::vector<int64_t> ptr(M.F + 1);
        std::vector<int32_t> list(nd.n);
        BIE_HIP(hipMemcpyAsync(ptr.data(), nd.ptr, ptr.size() * sizeof(int64_t), hipMemcpyDeviceToHost, s));
        BIE_HIP(hipMemcpyAsync(list.data(), nd.list, list.size() * sizeof(int32_t), hipMemcpyDeviceToHost, s));
        if (device_list) {
            Temp dr(size_t(M.F) * sizeof(int32_t));
            BIE_HIP(hipMemcpyAsync(dr.p, rank.data(), size_t(M.F) * sizeof(int32_t), hipMemcpyHostToDevice, s));
            op->flagged = pairs_of(nd, M.F, (const int32_t *)dr.p, s);
            BIE_HIP(hipStreamSynchronize(s));
        }
        BIE_HIP(hipStreamSynchronize(s));
        M.near.resize(2 * size_t(nd.n));
        for (int64_t p = 0; p < M.F; ++p)
            for (int64_t e = ptr[p]; e < ptr[p + 1]; ++e) {
                M.near[2 * e] = int32_t(p);
                M.near[2 * e + 1] = list[e];
            }
    } else if (device_list) {   // its matrix would take terabytes
        throw Error(BIE_ENOMEM, "no device holds a dense operator of " + std::to_string(M.F) + " triangles");
    }
}

void ranked_near(const bie_op *op, double near_factor, NearDev &out, hipStream_t s)
{
    const Mesh &M = op->mesh;
    const std::vector<int32_t> &rank = op->tri.rank;
    if (near_on_device(M.F)) {
        std::vector<int32_t> order(M.F);
        for (int64_t t = 0; t < M.F; ++t) order[rank[t]] = int32_t(t);
        near_search(M, near_factor, &order, out, s);
        return;
    }
    out.n = int64_t(M.near.size() / 2);
    std::vector<std::pair<int32_t, int32_t>> fl(out.n);
    for (int64_t i = 0; i < out.n; ++i) {
        const int32_t p = rank[M.near[2 * i]], q = rank[M.near[2 * i + 1]];
        fl[i] = { std::min(p, q), std::max(p, q) };
    }
    std::sort(fl.begin(), fl.end());
    std::vector<int64_t> ptr(M.F + 1, 0);
    std::vector<int32_t> list(out.n);
    for (int64_t i = 0; i < out.n; ++i) {
        ++ptr[fl[i].first + 1];
        list[i] = fl[i].second;
    }
    for (int64_t t = 0; t < M.F; ++t) ptr[t + 1] += ptr[t];
    BIE_HIP(device_malloc(&out.ptr, ptr.size() * sizeof(int64_t)));
    BIE_HIP(device_malloc(&out.list, std::max<size_t>(list.size(), 1) * sizeof(int32_t)));
    BIE_HIP(hipMemcpy(out.ptr, ptr.data(), ptr.size() * sizeof(int64_t), hipMemcpyHostToDevice));
    BIE_HIP(hipMemcpy(out.list, list.data(), list.size() * sizeof(int32_t), hipMemcpyHostToDevice));
}

int32_t *near_list(const NearDev &nd, int64_t F, hipStream_t s) { return pairs_of(nd, F, nullptr, s); }

}  // namespace bie
