// Exchanges between the lanes of a wave in registers (a permute through LDS takes its
// latency and its bandwidth for every 4 bytes), shared by the Krylov passes and the packed
// products.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

namespace bie {

template <int CTRL, int BANKS = 0xf> __device__ inline int dpp(int old, int v)
{
    return __builtin_amdgcn_update_dpp(old, v, CTRL, 0xf, BANKS, false);
}
template <int CTRL, int BANKS = 0xf> __device__ inline int2 dpp(int2 old, int2 v)
{
    return make_int2(dpp<CTRL, BANKS>(old.x, v.x), dpp<CTRL, BANKS>(old.y, v.y));
}
// a of lane and lane ^ O in the lanes whose bit O is clear, b in the others, added
template <int O> __device__ inline float pair_add(float a, float b)
{
    const int x = __builtin_bit_cast(int, a), y = __builtin_bit_cast(int, b);
    const auto s = O == 32 ? __builtin_amdgcn_permlane32_swap(x, y, false, false)
                           : __builtin_amdgcn_permlane16_swap(x, y, false, false);
    return __builtin_bit_cast(float, int(s[0])) + __builtin_bit_cast(float, int(s[1]));
}
template <int O> __device__ inline double pair_add(double a, double b)
{
    const int2 x = __builtin_bit_cast(int2, a), y = __builtin_bit_cast(int2, b);
    const auto lo = O == 32 ? __builtin_amdgcn_permlane32_swap(x.x, y.x, false, false)
                            : __builtin_amdgcn_permlane16_swap(x.x, y.x, false, false);
    const auto hi = O == 32 ? __builtin_amdgcn_permlane32_swap(x.y, y.y, false, false)
                            : __builtin_amdgcn_permlane16_swap(x.y, y.y, false, false);
    return __builtin_bit_cast(double, make_int2(int(lo[0]), int(hi[0]))) +
           __builtin_bit_cast(double, make_int2(int(lo[1]), int(hi[1])));
}
// the value of lane ^ O
template <int O, typename T> __device__ inline T lane_xor(T v)
{
    typedef std::conditional_t<sizeof(T) == 8, int2, int> W;
    const W w = __builtin_bit_cast(W, v), z{};
    W r;
    if (O == 8) r = dpp<0x128>(z, w);                                 // rotation of 16 lanes by 8
    else if (O == 4) r = dpp<0x114, 0xa>(dpp<0x104, 0x5>(z, w), w);   // shifts of 16 lanes by 4, for every other quad
    else if (O == 2) r = dpp<0x4e>(z, w);
    else r = dpp<0xb1>(z, w);
    return __builtin_bit_cast(T, r);
}

// Sums 8 complex values over a wave: each exchange halves what a lane carries (4 + 2 + 1
// exchanges, then 3 plain steps).  pr[0], pi[0] of lane L end with the total of
// value (L >> 3) & 7.
template <typename T>
__device__ inline void wave_sum8(T pr[8], T pi[8])
{
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        pr[i] = pair_add<32>(pr[i], pr[i + 4]);
        pi[i] = pair_add<32>(pi[i], pi[i + 4]);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        pr[i] = pair_add<16>(pr[i], pr[i + 2]);
        pi[i] = pair_add<16>(pi[i], pi[i + 2]);
    }
    const bool b = threadIdx.x & 8;
    const T sr = b ? pr[0] : pr[1], si = b ? pi[0] : pi[1];
    const T kr = b ? pr[1] : pr[0], ki = b ? pi[1] : pi[0];
    pr[0] = kr + lane_xor<8>(sr);
    pi[0] = ki + lane_xor<8>(si);
    pr[0] += lane_xor<4>(pr[0]);
    pi[0] += lane_xor<4>(pi[0]);
    pr[0] += lane_xor<2>(pr[0]);
    pi[0] += lane_xor<2>(pi[0]);
    pr[0] += lane_xor<1>(pr[0]);
    pi[0] += lane_xor<1>(pi[0]);
}

}  // namespace bie
