// Small helpers of the step kernels.
#pragma once
#include "fm_device.h"

template <typename T>
__global__ void k_convert(const float* __restrict__ src, T* __restrict__ dst, long n) {
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x)
    Store<T>::st(dst + i, src[i]);
}

// Greedy choice: lowest index among exact ties
__device__ __forceinline__ void argmax_merge(float& bv, int& bi, float v, int i) {
  if (v > bv || (v == bv && i < bi)) { bv = v; bi = i; }
}
