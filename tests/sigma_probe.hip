// The branch-free forms of sigma and the library's (sigma.h, common.h) on arrays, for test_gpu_sigma.py.
#include "common.h"
#include "sigma.h"

namespace {
template <int ACT> __global__ void sigma32_kernel(const float* z, float* flat, float* lib, long n) {
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    flat[i] = act_flat<ACT>(z[i]);
    lib[i] = td_act(z[i], ACT);
}
template <int ACT> __global__ void sigma64_kernel(const double* z, double* flat, double* lib, long n) {
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    flat[i] = act_flat_f64<ACT>(z[i]);
    lib[i] = td_act_f64(z[i], ACT);
}
}  // namespace

extern "C" int sigma_probe(int act, int bits, const void* z, void* flat, void* lib, long n) {
    const dim3 grid((unsigned)((n + 255) / 256));
    auto f32 = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(256), 0, 0, (const float*)z, (float*)flat, (float*)lib, n); };
    auto f64 = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, dim3(256), 0, 0, (const double*)z, (double*)flat, (double*)lib, n); };
    if (n < 1 || (bits != 32 && bits != 64)) return 1;
    if (act == TARDIS_ACT_GELU_ERF) bits == 32 ? f32(sigma32_kernel<TARDIS_ACT_GELU_ERF>) : f64(sigma64_kernel<TARDIS_ACT_GELU_ERF>);
    else if (act == TARDIS_ACT_GELU_TANH) bits == 32 ? f32(sigma32_kernel<TARDIS_ACT_GELU_TANH>) : f64(sigma64_kernel<TARDIS_ACT_GELU_TANH>);
    else return 1;
    return hipDeviceSynchronize() != hipSuccess || hipGetLastError() != hipSuccess;
}
