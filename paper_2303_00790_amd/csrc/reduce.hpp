// Deterministic sums over a wave, a workgroup and a launch's partials.
#pragma once
#include <hip/hip_runtime.h>

namespace chf {

__device__ inline double wave_sum(double v) {
    for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off, 64);
    return v;
}

// sum over the workgroup, the same on all threads; sh holds one value per wave
__device__ inline double group_sum(double v, double* sh) {
    v = wave_sum(v);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    double s = 0.0;
    for (unsigned w = 0; w < blockDim.x / 64; ++w) s += sh[w];
    return s;
}

// sum of n partials by one workgroup: every workgroup of a launch that needs
// the sum forms it, in the same order
__device__ inline double parts_sum(const double* part, int n, double* sh) {
    double v = 0.0;
    for (int i = threadIdx.x; i < n; i += blockDim.x) v += part[i];
    return group_sum(v, sh);
}

}  // namespace chf
