// Cross-lane moves and sums by DPP, without the LDS round trips of shuffles.
#pragma once

#include <hip/hip_runtime.h>

namespace mls {

template <int CTRL, int ROWS = 0xf>
__device__ __forceinline__ float dpp(float v)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, ROWS, 0xf, ROWS == 0xf));
}
template <int CTRL, int ROWS = 0xf>
__device__ __forceinline__ double dpp(double v)
{
    const long long u = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)u, CTRL, ROWS, 0xf, ROWS == 0xf);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(u >> 32), CTRL, ROWS, 0xf, ROWS == 0xf);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}
// the value of lane - 1 (lane 0: zero) and of lane + 1 (lane 63: zero)
template <typename T>
__device__ __forceinline__ T west(T v) { return dpp<0x138>(v); }
template <typename T>
__device__ __forceinline__ T east(T v) { return dpp<0x130>(v); }

// sum over the wave in lane 63: within rows of 16, then across the rows
__device__ __forceinline__ double lane63_sum(double v)
{
    v += dpp<0x111>(v);
    v += dpp<0x112>(v);
    v += dpp<0x114>(v);
    v += dpp<0x118>(v);
    v += dpp<0x142, 0xa>(v);
    v += dpp<0x143, 0xc>(v);
    return v;
}
__device__ __forceinline__ double read_lane(double v, int lane)
{
    const long long u = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)u, lane), hi = __builtin_amdgcn_readlane((int)(u >> 32), lane);
    return __longlong_as_double(((long long)hi << 32) | (unsigned)lo);
}

}  // namespace mls
