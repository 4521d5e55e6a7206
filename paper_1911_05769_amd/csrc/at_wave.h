// Exchange between the lanes of a wave64 without a barrier.
#pragma once

#include <hip/hip_runtime.h>

namespace atk {

namespace {

// Lanes of a wave see each other's LDS writes in program order; this only
// keeps the compiler from moving accesses across
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// the value of the lane to the left (lane - 1) / right (lane + 1); `end` at
// the wave's end
template <int CTRL, bool END>
__device__ __forceinline__ double dpp_shift(double end, double x)
{
    const long long b = __double_as_longlong(x), e = __double_as_longlong(end);
    int lo, hi;
    if constexpr (END) {
        lo = __builtin_amdgcn_update_dpp((int)e, (int)b, CTRL, 0xf, 0xf, false);
        hi = __builtin_amdgcn_update_dpp((int)(e >> 32), (int)(b >> 32), CTRL, 0xf, 0xf, false);
    } else {
        lo = __builtin_amdgcn_mov_dpp((int)b, CTRL, 0xf, 0xf, true);
        hi = __builtin_amdgcn_mov_dpp((int)(b >> 32), CTRL, 0xf, 0xf, true);
    }
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
template <bool END>
__device__ __forceinline__ double from_left(double end, double x) { return dpp_shift<0x138, END>(end, x); }
template <bool END>
__device__ __forceinline__ double from_right(double end, double x) { return dpp_shift<0x130, END>(end, x); }

}  // namespace

}  // namespace atk
