// Exchanges between the lanes of a wave, and the leftmost minimum of (value,
// index) pairs.
#pragma once

#include "common.h"

namespace gpic {
namespace {

// Leftmost-argmin merge of (value, index) pairs.
__device__ __forceinline__ void amin_merge(double &b, int64_t &a, double ob,
                                           int64_t oa)
{
    if (ob < b || (ob == b && oa < a)) {
        b = ob;
        a = oa;
    }
}

// The value of lane (lane xor K): data-parallel moves for K = 1, 2, 8
// (quad permutations, a rotation by 8 within a row of 16), swizzles for
// K = 4, 16, a permute for K = 32.
template <int K>
__device__ __forceinline__ int lane_xor(int x)
{
    if (K == 1)
        return __builtin_amdgcn_mov_dpp(x, 0xb1, 0xf, 0xf, false);
    if (K == 2)
        return __builtin_amdgcn_mov_dpp(x, 0x4e, 0xf, 0xf, false);
    if (K == 4)
        return __builtin_amdgcn_ds_swizzle(x, 0x101f);
    if (K == 8)
        return __builtin_amdgcn_mov_dpp(x, 0x128, 0xf, 0xf, false);
    if (K == 16)
        return __builtin_amdgcn_ds_swizzle(x, 0x401f);
    return __shfl_xor(x, 32, kWave);
}

template <int K>
__device__ __forceinline__ double lane_xor(double x)
{
    const long long b = __double_as_longlong(x);
    const int lo = lane_xor<K>((int)(b & 0xffffffffll));
    const int hi = lane_xor<K>((int)(b >> 32));
    return __longlong_as_double(((long long)(unsigned)hi << 32) | (long long)(unsigned)lo);
}

template <int K>
__device__ __forceinline__ void argmin_step(double &best, int32_t &arg)
{
    const double ob = lane_xor<K>(best);
    const int32_t oa = lane_xor<K>(arg);
    if (ob < best || (ob == best && oa < arg)) {
        best = ob;
        arg = oa;
    }
}

// Leftmost minimum of (value, index) over the wave, in every lane (an
// index of INT64_MAX, no candidate, travels as INT32_MAX).
__device__ __forceinline__ void wave_argmin(double &best, int64_t &arg)
{
    int32_t a = (arg == INT64_MAX) ? INT32_MAX : (int32_t)arg;
    argmin_step<32>(best, a);
    argmin_step<16>(best, a);
    argmin_step<8>(best, a);
    argmin_step<4>(best, a);
    argmin_step<2>(best, a);
    argmin_step<1>(best, a);
    arg = (a == INT32_MAX) ? INT64_MAX : (int64_t)a;
}

} // namespace
} // namespace gpic
