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

// 0.5 x (1 + tanh(u)) = x / (1 + exp(-2u)): nothing cancels where tanh comes near -1, and it is two instructions of the transcendental unit in
// place of the library's tanh (whose sum with 1 is off by 2^-24 of 1, of 0.005 at u = -3).
__device__ __forceinline__ float gelu_tanh_f(float x) {
  const float k = 0.7978845608028654f;  // sqrt(2/pi)
  const float u = k * (x + 0.044715f * x * x * x);
  return x * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(u * -2.8853900817779268f));      // 2 log2(e)
}
// 1 / sqrt(x) of a normal x: the unit's estimate and one Newton step, a chain of 5 in place of the 25 of a correctly rounded root and quotient
__device__ __forceinline__ float rsqrt_f(float x) {
  const float r = __builtin_amdgcn_rsqf(x);
  return fmaf(r * 0.5f, fmaf(-x * r, r, 1.0f), r);
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
