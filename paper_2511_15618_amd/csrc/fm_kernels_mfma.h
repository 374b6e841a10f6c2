// Layouts of weights, activations and K/V caches in matrix-operand order (gfx950) and what puts data into them; agent-scope access for
// exchanges inside a launch.
//
// MFMA 16x16x32 f16 operand layout (lane l of 64):
//   A[16 x 32]: row l%16, k = (l/16)*8 .. +8      B[32 x 16]: col l%16, k = (l/16)*8 .. +8
//   C[16 x 16]: col l%16, rows (l/16)*4 + i, i = 0..3
// The fp32 path uses the same layouts with eight floats in the place of eight halves: component j of the eight is one 16x16x4 f32
// MFMA (A: row l%16, k = l/16), i.e. the eight of them sum over the same 32 k.
#pragma once
#include <type_traits>
#include "fm_device.h"

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));

// operands of a storage type: a lane's eight k values, four neighbouring columns, and the product over 32 k
template <typename T> struct Op;
template <> struct Op<f16_t> {
  typedef f16x8 V8;
  typedef f16x4 V4;
  static __device__ __forceinline__ f32x4 mul(const V8& a, const V8& b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0); }
};
template <> struct Op<float> {
  typedef f32x8 V8;
  typedef f32x4 V4;
  static __device__ __forceinline__ f32x4 mul(const V8& a, const V8& b, f32x4 c) {
#pragma unroll
    for (int j = 0; j < 8; j++) c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[j], b[j], c, 0, 0, 0);
    return c;
  }
};

// Values of neighbouring lanes without the trip to LDS that a shuffle is (ds_bpermute, about 100 cycles in a serial chain).
// (The decode kernels' maxima and sums with these instead of shuffles, the same results: a step of 24 blocks at d = 768 and three
// sequences 1212 -> 1193 us, the first blocks of two new sequences 1258 -> 1237 us.)
// Rows are the 16 lanes of equal lane / 16.
template <int CTRL> __device__ __forceinline__ float lane_dpp(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, true));
}
__device__ __forceinline__ float lane_xor1(float v) { return lane_dpp<0xB1>(v); }        // quad_perm [1, 0, 3, 2]
__device__ __forceinline__ float lane_xor8(float v) { return lane_dpp<0x128>(v); }       // row_ror 8
__device__ __forceinline__ float row16_sum(float v) {      // sum over a row, in each of its lanes
  v += lane_dpp<0xB1>(v);
  v += lane_dpp<0x4E>(v);        // quad_perm [2, 3, 0, 1]
  v += lane_dpp<0x141>(v);       // row_half_mirror
  v += lane_dpp<0x140>(v);       // row_mirror
  return v;
}
__device__ __forceinline__ int row16_max(int v) {          // the same steps, maximum
  v = max(v, __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, true));
  v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, true));
  v = max(v, __builtin_amdgcn_update_dpp(0, v, 0x141, 0xF, 0xF, true));
  return max(v, __builtin_amdgcn_update_dpp(0, v, 0x140, 0xF, 0xF, true));
}
__device__ __forceinline__ float lane_xor32(float v) {     // the other half of the wave
  const auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float((threadIdx.x & 32) ? a[0] : a[1]);
}
// sum and maximum over the four rows, lane by lane, in each of them (the same results as with shuffles by 16 and 32)
__device__ __forceinline__ float rows_sum(float v) {
  const unsigned u = __float_as_uint(v);
  const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  const float w = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(w), __float_as_uint(w), false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}
__device__ __forceinline__ float rows_max(float v) {
  const unsigned u = __float_as_uint(v);
  const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  const float w = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(w), __float_as_uint(w), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}

// Greedy choice over a wave: the largest value, among equals the lowest index; in every lane
__device__ __forceinline__ void wave_argmax(float& bv, int& bi) {
  float m = fmaxf(bv, lane_dpp<0xB1>(bv));
  m = fmaxf(m, lane_dpp<0x4E>(m));
  m = fmaxf(m, lane_dpp<0x141>(m));
  m = rows_max(fmaxf(m, lane_dpp<0x140>(m)));
  int i = bv == m ? bi : 0x7fffffff;
  i = min(i, __builtin_amdgcn_update_dpp(0, i, 0xB1, 0xF, 0xF, true));
  i = min(i, __builtin_amdgcn_update_dpp(0, i, 0x4E, 0xF, 0xF, true));
  i = min(i, __builtin_amdgcn_update_dpp(0, i, 0x141, 0xF, 0xF, true));
  i = min(i, __builtin_amdgcn_update_dpp(0, i, 0x140, 0xF, 0xF, true));
  const auto a = __builtin_amdgcn_permlane16_swap((unsigned)i, (unsigned)i, false, false);
  i = min((int)a[0], (int)a[1]);
  const auto b = __builtin_amdgcn_permlane32_swap((unsigned)i, (unsigned)i, false, false);
  bv = m;
  bi = min((int)b[0], (int)b[1]);
}

// Values that workgroups of one launch hand to each other (attention parts) are written and read at agent scope: the stores are
// written through to where all dies see them, the loads bypass the die's own L2.
__device__ __forceinline__ void st_agent(float* p, float v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// The loads come as buffer loads (byte offset `o` into `bytes` from a uniform base, 0 beyond them): the compiler knows them, so it keeps many in
// flight where atomic loads would go one by one, and places every wait itself.  It may also take two of them for one, or move them: a loop
// that polls has a compiler barrier (agent_again) in front of them, and so has a batch that is to leave together behind it.
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
typedef __amdgpu_buffer_rsrc_t agent_buf_t;
__device__ __forceinline__ agent_buf_t agent_buf(const void* base, int bytes) { return __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, bytes, 0x00027000); }
__device__ __forceinline__ u32x4 ld_agent4(agent_buf_t b, int o) { return __builtin_amdgcn_raw_buffer_load_b128(b, o, 0, 16); }      // 16: sc1
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ u32x2 ld_agent2(agent_buf_t b, int o) { return __builtin_amdgcn_raw_buffer_load_b64(b, o, 0, 16); }
__device__ __forceinline__ unsigned ld_agent1(agent_buf_t b, int o) { return __builtin_amdgcn_raw_buffer_load_b32(b, o, 0, 16); }
__device__ __forceinline__ void agent_again() { asm volatile("" ::: "memory"); }

// ------------------------------------------------------------------------------------------
// Cache layouts: one 32-key block of a head = 32 HD values (4 KiB of halves for the 64-wide heads
// of the benchmark configurations; HD = 96 and 128 are the paper's own model shapes)
// ------------------------------------------------------------------------------------------
// K: HD/16 A-fragments per block, fragment f = (key/16)*(HD/32) + dim/32, lane = key%16 + 16*((dim%32)/8)
template <int HD = 64>
__device__ __forceinline__ long kblk_off(int key, int dim) {
  const int r = key & 31;
  const int f = (r >> 4) * (HD / 32) + (dim >> 5);
  const int lane = (r & 15) + 16 * ((dim & 31) >> 3);
  return (long)(key >> 5) * (32 * HD) + (f * 64 + lane) * 8 + (dim & 7);
}
// V: transposed inside the block, [dim][slot]; slot order matches the C-layout of the score tile so
// that the probabilities never leave registers: key r -> g = (r%16)/4, slot = g*8 + (r/16)*4 + r%4
template <int HD = 64>
__device__ __forceinline__ long vblk_off(int key, int dim) {
  const int r = key & 31;
  const int slot = ((r & 15) >> 2) * 8 + (r >> 4) * 4 + (r & 3);
  return (long)(key >> 5) * (32 * HD) + dim * 32 + slot;
}

// fp32 key rows and value rows [M][ld] of a condition memory -> blocked caches (a null pair: not in this call)
template <typename T, int HD>
__global__ void k_mem_kv_store(const float* __restrict__ k, const float* __restrict__ v, int ld, T* __restrict__ Kc, T* __restrict__ Vc, int H,
                                 int M, int capb) {
  const int m = blockIdx.x;
  const int d = H * HD;
  for (int i = threadIdx.x; i < d; i += blockDim.x) {
    const int hh = i / HD, e = i % HD;
    const long base = (long)hh * capb * (32 * HD);
    if (k) Kc[base + kblk_off<HD>(m, e)] = (T)k[(long)m * ld + i];
    if (v) Vc[base + vblk_off<HD>(m, e)] = (T)v[(long)m * ld + i];
  }
}

// A lane's part of fragment (nt, kt) of a matrix [N][K] fp32: W[nt*16 + l%16][kt*32 + (l/16)*8 + j] in the storage type, rows past N zero.
// rope_rows > 0 (projections to queries and keys): rows below it belong to heads of width hd whose rotary pairs (i, i + hd/2)
// must meet in one result tile: tile q of a head holds dims q*8..+8 and hd/2 + q*8..+8, i.e. both halves of 8 pairs.
template <typename T>
__device__ __forceinline__ typename Op<T>::V8 tile_part(const float* __restrict__ src, int N, int K, int nt, int kt, int lane, int rope_rows, int hd) {
  typedef float f32x8u __attribute__((ext_vector_type(8), aligned(4)));      // a caller's tensor is aligned to its elements, no more
  int n = nt * 16 + (lane & 15);
  if (n < rope_rows) {
    const int hh = n / hd, qd = (n % hd) >> 4, c = n & 15;
    n = hh * hd + (c < 8 ? qd * 8 + c : hd / 2 + qd * 8 + (c - 8));
  }
  const f32x8u v = *reinterpret_cast<const f32x8u*>(src + (long)min(n, N - 1) * K + kt * 32 + (lane >> 4) * 8);
  typename Op<T>::V8 o;
#pragma unroll
  for (int j = 0; j < 8; j++) o[j] = n < N ? (T)v[j] : (T)0.f;
  return o;
}
// weights [N][K] fp32 -> storage type (half: bf16-valued, exact), tiled
template <typename T>
__global__ void k_tile_weight(const float* __restrict__ src, T* __restrict__ dst, int N, int K, int Npad, int rope_rows, int hd) {
  const long total = (long)Npad * K / 8;
  const int KT = K / 32;
  for (long v = blockIdx.x * (long)blockDim.x + threadIdx.x; v < total; v += (long)gridDim.x * blockDim.x) {
    const long frag = v >> 6;
    *reinterpret_cast<typename Op<T>::V8*>(dst + v * 8) = tile_part<T>(src, N, K, (int)(frag / KT), (int)(frag % KT), (int)(v & 63), rope_rows, hd);
  }
}
