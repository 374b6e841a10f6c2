// Device-side helpers shared by the kernels: storage-type traits, conversion, reductions.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

// Storage / MFMA operand type of the "bf16" configurations.  Their weights are bf16-valued, which
// convert to IEEE half exactly (8-bit significand into 11 bits; only magnitudes below 2^-14 go
// subnormal), and half keeps 3 more significand bits for activations and K/V at the same byte
// and MFMA cost, which is what holds the logits inside the stated tolerance.
typedef _Float16 f16_t;

template <typename T> struct Store;
template <> struct Store<float> {
  static __device__ __forceinline__ float ld(const float* p) { return *p; }
  static __device__ __forceinline__ void st(float* p, float v) { *p = v; }
};
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
template <> struct Store<f16_t> {
  static __device__ __forceinline__ float ld(const f16_t* p) { return (float)*p; }
  static __device__ __forceinline__ void st(f16_t* p, float v) { *p = (f16_t)v; }   // round-to-nearest-even
};

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
  return v;
}
__device__ __forceinline__ float wave_max(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
  return v;
}

// The library's tanh.  Largest error against float64 for x ~ N(0, 1) 3.7e-7, rms 2.4e-8; as x / (1 + exp(-2u)) from the transcendental unit's exp2 and reciprocal,
// which is two instructions, 4.5e-7 and 3.1e-8 (steps of d = 512 562 us instead of 569, of d = 1024 1445 instead of 1453, both with the reciprocal
// root of the norms from the unit too).
__device__ __forceinline__ float gelu_tanh_f(float x) {
  const float k = 0.7978845608028654f;  // sqrt(2/pi)
  float u = k * (x + 0.044715f * x * x * x);
  return 0.5f * x * (1.0f + tanhf(u));
}

template <typename T>
__global__ void k_convert(const float* __restrict__ src, T* __restrict__ dst, long n) {
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x)
    Store<T>::st(dst + i, src[i]);
}

// Greedy choice: lowest index among exact ties
__device__ __forceinline__ void argmax_merge(float& bv, int& bi, float v, int i) {
  if (v > bv || (v == bv && i < bi)) { bv = v; bi = i; }
}
