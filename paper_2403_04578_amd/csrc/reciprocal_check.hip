// The sweeps' reciprocals (device_math.h) of an array, for the tests that compare them with the
// division.  Not part of the API: include/tpf.h does not declare it.
#include "device_math.h"
#include "tpf_internal.h"

namespace {

template <typename R>
__global__ __launch_bounds__(256) void reciprocals_kernel(const R *__restrict__ x, R *__restrict__ y, long long count) {
    const long long k = (long long)blockIdx.x * 256 + threadIdx.x;
    if (k >= count) return;
    if constexpr (sizeof(R) == 8)
        y[k] = tpf::reciprocal(x[k]);
    else
        y[k] = tpf::reciprocal32(x[k]);
}

}  // namespace

// x, y: device arrays of `count` doubles (f64) or floats, count up to 2^30.
extern "C" int tpf_check_reciprocals(const void *x, void *y, int64_t count, int f64, hipStream_t stream) {
    if (!x || !y || count < 1 || count > (1 << 30)) return tpf::fail(TPF_ERR_INVALID_ARG, "1 to 2^30 values");
    const dim3 grid((unsigned)((count + 255) / 256));
    if (f64)
        hipLaunchKernelGGL(reciprocals_kernel<double>, grid, dim3(256), 0, stream, (const double *)x, (double *)y,
                           (long long)count);
    else
        hipLaunchKernelGGL(reciprocals_kernel<float>, grid, dim3(256), 0, stream, (const float *)x, (float *)y,
                           (long long)count);
    return hipGetLastError() == hipSuccess ? TPF_OK : tpf::fail(TPF_ERR_DEVICE, "launch failed");
}
