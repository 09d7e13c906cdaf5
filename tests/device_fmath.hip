// The binary32 pair of csrc/fmath.hpp as the particle kernels compile it, over a
// range of the generator's arguments a = k 2^-24 (test_gpu_fmath.py).
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fmath.hpp"

__global__ void __launch_bounds__(256) k_terms(uint32_t k0, uint32_t n, float* ln, float* radius, float* sn, float* cs) {
    const uint32_t i = blockIdx.x * 256u + threadIdx.x;
    if (i >= n) return;
    const float a = (float)(k0 + i) * 0x1p-24f;
    ln[i] = lbmpcd::ln_unit32(1.0f - a);
    radius[i] = lbmpcd::root32(-2.0f * lbmpcd::ln_unit32(1.0f - a));
    lbmpcd::sincos_2pi32(a, &sn[i], &cs[i]);
}

extern "C" int device_terms(uint32_t k0, uint32_t n, float* ln, float* radius, float* sn, float* cs, void* stream) {
    hipLaunchKernelGGL(k_terms, dim3((n + 255u) / 256u), dim3(256), 0, (hipStream_t)stream, k0, n, ln, radius, sn, cs);
    return (int)hipGetLastError();
}
