// dpp.h -- values of neighbouring lanes of a wave (DPP wave shifts).
#pragma once

#include <hip/hip_runtime.h>

namespace lbm {

// The value of the lane to the left (wave_shr:1) / right (wave_shl:1); the
// first / last lane gets 0 (its results are never written).
template <int CTRL> __device__ __forceinline__ unsigned lane_shift(unsigned v)
{
    return (unsigned)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, true);
}
template <int CTRL> __device__ __forceinline__ float lane_shift(float v)
{
    return __builtin_bit_cast(float, lane_shift<CTRL>(__builtin_bit_cast(unsigned, v)));
}
template <int CTRL> __device__ __forceinline__ double lane_shift(double v)
{
    const unsigned long long b = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = lane_shift<CTRL>((unsigned)b), hi = lane_shift<CTRL>((unsigned)(b >> 32));
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}
template <class C> __device__ __forceinline__ C from_left(C v) { return lane_shift<0x138>(v); }
template <class C> __device__ __forceinline__ C from_right(C v) { return lane_shift<0x130>(v); }

}  // namespace lbm
