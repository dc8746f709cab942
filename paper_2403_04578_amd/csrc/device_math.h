// Reciprocals of the sweep kernels and a barrier for LDS alone.
#pragma once

#include <hip/hip_runtime.h>

namespace tpf {
namespace {

// 1 / x for a finite positive x: the hardware estimate (within 2^-23) and two Newton steps, which
// leave 2^-92 before the last rounding: the division's result but for one x in about 2^38 (none
// differs among 2^24 at each of seven exponents, tests/test_gpu_reciprocals.py).  The compiler's
// division spends eleven vector instructions where this takes five.
__device__ __forceinline__ double reciprocal(double x) {
    double y = __builtin_amdgcn_rcp(x);
    y = __builtin_fma(__builtin_fma(-x, y, 1.0), y, y);
    return __builtin_fma(__builtin_fma(-x, y, 1.0), y, y);
}

// 1 / x, correctly rounded, for x from 1e-30 to 2^125: the hardware estimate and one Newton
// step, equal to the division for every mantissa (all compared at eight exponents,
// tests/test_gpu_reciprocals.py) at three instructions instead of ten.  Beyond, where an iterate has diverged and the injection
// vanishes against any voltage, the estimate itself (0 for inf).
__device__ __forceinline__ float reciprocal32(float x) {
    const float y = __builtin_amdgcn_rcpf(x);
    return x < 0x1p125f ? __builtin_fmaf(__builtin_fmaf(-x, y, 1.0f), y, y) : y;
}

// A barrier for data exchanged in LDS alone: it waits for this wave's LDS accesses, not for its
// global ones, so that the operands requested ahead and the results on their way out stay in
// flight across it (__syncthreads drains both, an L2 round trip each time).
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

}  // namespace
}  // namespace tpf
