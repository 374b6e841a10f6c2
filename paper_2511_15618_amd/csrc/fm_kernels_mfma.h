// Half-precision MFMA kernels for gfx950 (64-wide wavefronts, v_mfma_f32_16x16x32_f16).
//
//  * k_gemm_mfma : skinny weight-streaming GEMM.  Weights are pre-tiled at load time into MFMA
//                  B-operand order so that every wave load is one contiguous 1 KiB burst; the four
//                  waves of a workgroup split K and reduce through LDS in a fixed order.  K is not
//                  split across workgroups: publishing partial sums inside a launch needs an
//                  agent-scope release fence, which costs more than the parallelism gains here.
//  * k_attn_mfma : block attention over a K/V cache (flash-decoding): fixed key ranges split across
//                  workgroups and waves, online softmax in fp32, P kept in registers between the two
//                  MFMAs by storing V in a blocked, slot-permuted transposed layout; partial results
//                  merged in range order (in the launch, or by k_attn_merge when there are many).
//
// MFMA 16x16x32 operand layout (lane l of 64):
//   A[16 x 32]: row l%16, k = (l/16)*8 .. +8      B[32 x 16]: col l%16, k = (l/16)*8 .. +8
//   C[16 x 16]: col l%16, rows (l/16)*4 + i, i = 0..3
#pragma once
#include <type_traits>
#include "fm_device.h"
#include "fm_kernels_basic.h"

typedef float f32x4 __attribute__((ext_vector_type(4)));

// Cross-workgroup exchange inside one launch (split-KV partials): values are written and read with
// agent-scope atomics and published with an agent-scope RELEASE fence before the arrival counter is
// bumped.  A workgroup-scope fence is not enough on this chip: the write-through of an agent-scope store
// can still be in flight when the counter increment lands, and the last arriver then reads the previous
// launch's data (seen as run-to-run differences in one token per ~10^4 steps).  The consumer side needs
// no invalidate because it reads the partials with agent-scope loads.
__device__ __forceinline__ void st_agent(float* p, float v) {
  __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ float ld_agent(const float* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void publish_fence() { __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent"); }

// ------------------------------------------------------------------------------------------
// Cache layouts of the half-precision path: one 32-key block of a head = 32 HD halves (4 KiB for the 64-wide heads
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

template <int HD>
__global__ void k_mem_kv_store_h(const float* __restrict__ kv, f16_t* __restrict__ Kc, f16_t* __restrict__ Vc, int H,
                                 int M, int capb) {
  const int m = blockIdx.x;
  const int d = H * HD;
  for (int i = threadIdx.x; i < d; i += blockDim.x) {
    const int hh = i / HD, e = i % HD;
    const long base = (long)hh * capb * (32 * HD);
    Kc[base + kblk_off<HD>(m, e)] = (f16_t)kv[(long)m * 2 * d + i];
    Vc[base + vblk_off<HD>(m, e)] = (f16_t)kv[(long)m * 2 * d + d + i];
  }
}

// weights [N][K] fp32 (bf16-valued) -> half, tiled: fragment (nt, kt) holds W[nt*16 + l%16][kt*32 + (l/16)*8 + j]
// rope_rows > 0 (projections to queries and keys): rows below it belong to heads of width hd whose rotary pairs (i, i + hd/2)
// must meet in one result tile: tile q of a head holds dims q*8..+8 and hd/2 + q*8..+8, i.e. both halves of 8 pairs.
__global__ void k_tile_weight(const float* __restrict__ src, f16_t* __restrict__ dst, int N, int K, int Npad, int rope_rows, int hd) {
  const long total = (long)Npad * K / 8;
  for (long v = blockIdx.x * (long)blockDim.x + threadIdx.x; v < total; v += (long)gridDim.x * blockDim.x) {
    const int lane = (int)(v & 63);
    const long frag = v >> 6;
    const int KT = K / 32;
    const int kt = (int)(frag % KT), nt = (int)(frag / KT);
    int n = nt * 16 + (lane & 15);
    const int k = kt * 32 + (lane >> 4) * 8;
    if (n < rope_rows) {
      const int hh = n / hd, qd = (n % hd) >> 4, c = n & 15;
      n = hh * hd + (c < 8 ? qd * 8 + c : hd / 2 + qd * 8 + (c - 8));
    }
    f16x8 o;
#pragma unroll
    for (int j = 0; j < 8; j++) o[j] = n < N ? (f16_t)src[(long)n * K + k + j] : (f16_t)0.f;
    *reinterpret_cast<f16x8*>(dst + v * 8) = o;
  }
}

// ------------------------------------------------------------------------------------------
// GEMM
// ------------------------------------------------------------------------------------------
// The wave index is made provably wave-uniform (readfirstlane) in every MFMA kernel: MFMA ignores the EXEC mask,
// so an MFMA guarded by a condition the compiler takes for divergent would run on a false guard as well.
struct GemmSplit {
  int kt_per_wave;   // K fragments (of 32) each wave walks
};

// NORM: X is fp32 and each row is RMS-normalised on the fly: the MFMA runs on half(x * gain) and the per-row factor
// 1/rms is applied to the accumulated tile (every workgroup walks the whole K of its rows, so it has the row sums
// of squares itself; partial sums per wave meet in LDS next to the partial tiles, in a fixed order).
// (two workgroups per CU: launches of 257..512 workgroups, e.g. the 288 and 384 tiles of d = 1536, then take one
// round instead of two)
// NW waves per workgroup (4, 8 or 16) split K: launches with few column tiles (N = d gives 64 to 96 of them)
// take more waves per workgroup so that enough loads are in flight and each wave's K walk stays short.
// NC column tiles of 16 per workgroup (1 or 2): with two, an activation fragment loaded (and normalised) once feeds two
// MFMAs, which halves what the wide projections (N >= 2048) pull out of L2 for their activations.
template <int MT, int EPI, bool NORM, int NW, int NC = 1>
__global__ __launch_bounds__(NW * 64, NW == 4 ? 2 : 1) void k_gemm_mfma(GemmArgs a, GemmSplit sp) {
  if (a.run_flag && *a.run_flag == 0) return;
  static_assert(NW * MT * NC <= 60, "partial tiles of all waves must fit the static LDS limit");
  __shared__ f32x4 red[NW][MT * NC][64];
  __shared__ float sq[NORM ? NW : 1][MT][16];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int nt = blockIdx.x;
  const int nmb = (a.M + MT * 16 - 1) / (MT * 16);
  const int g = blockIdx.z / nmb, mb = blockIdx.z % nmb;
  const int KT = a.K / 32;
  typedef typename std::conditional<NORM, float, f16_t>::type XT;
  const XT* X = (const XT*)a.X + (long)g * a.gsx;
  const f16_t* W = (const f16_t*)a.W + (long)g * a.gsw + ((long)nt * NC * KT) * 512;   // column tile c of this workgroup: + c * KT * 512
  const int m0 = mb * MT * 16;
  // A-fragment row pointers (rows past M are clamped: computed, never stored)
  const XT* xrow[MT];
#pragma unroll
  for (int mt = 0; mt < MT; mt++) {
    int m = m0 + mt * 16 + (lane & 15);
    m = m < a.M ? m : a.M - 1;
    xrow[mt] = X + (long)m * a.ldx + (lane >> 4) * 8;
  }
  f32x4 acc[MT][NC];
  float ss[MT];
#pragma unroll
  for (int mt = 0; mt < MT; mt++) {
    ss[mt] = 0.f;
#pragma unroll
    for (int c = 0; c < NC; c++) acc[mt][c] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  const int kt0 = wave * sp.kt_per_wave;
  const int kt1 = min(kt0 + sp.kt_per_wave, KT);

  // K is walked in chunks of U fragments; the loads of the next chunk are in flight while this one is
  // multiplied (a workgroup is often alone on its CU, so nothing else would hide the latency)
  constexpr int U4 = NORM ? (MT <= 2 ? 4 : MT <= 5 ? 2 : 1) : (MT <= 2 ? 8 : MT <= 5 ? 4 : 2);
  constexpr int U = NW == 16 ? (U4 >= 4 ? U4 / 4 : 1) : NW == 8 ? (U4 >= 2 ? U4 / 2 : 1) : U4;
  struct AFrag { typename std::conditional<NORM, f32x4, f16x8>::type lo; f32x4 hi; };   // hi only used when NORM
  f16x8 bc[NC][U];
  AFrag ac[MT][U];
  f32x4 gc[NORM ? U : 1][2];
  const int nk = kt1 - kt0;
  auto kmap = [&](int i) { return kt0 + i; };
  auto load_chunk = [&](f16x8 (&b)[NC][U], AFrag (&af)[MT][U], f32x4 (&gg)[NORM ? U : 1][2], int i0) {
#pragma unroll
    for (int u = 0; u < U; u++) {
      if (i0 + u < nk) {
        const int kt = kmap(i0 + u);
#pragma unroll
        for (int c = 0; c < NC; c++) b[c][u] = *reinterpret_cast<const f16x8*>(W + ((long)(c * KT + kt) * 64 + lane) * 8);
        if constexpr (NORM) {
          const float* gp = a.gain + kt * 32 + (lane >> 4) * 8;
          gg[u][0] = *reinterpret_cast<const f32x4*>(gp);
          gg[u][1] = *reinterpret_cast<const f32x4*>(gp + 4);
        }
#pragma unroll
        for (int mt = 0; mt < MT; mt++) {
          if constexpr (NORM) {
            af[mt][u].lo = *reinterpret_cast<const f32x4*>(xrow[mt] + kt * 32);
            af[mt][u].hi = *reinterpret_cast<const f32x4*>(xrow[mt] + kt * 32 + 4);
          } else {
            af[mt][u].lo = *reinterpret_cast<const f16x8*>(xrow[mt] + kt * 32);
          }
        }
      }
    }
  };
  load_chunk(bc, ac, gc, 0);
  for (int i0 = 0; i0 < nk; i0 += U) {
    f16x8 bn[NC][U];
    AFrag an[MT][U];
    f32x4 gn[NORM ? U : 1][2];
    load_chunk(bn, an, gn, i0 + U);
#pragma unroll
    for (int u = 0; u < U; u++) {
      if (i0 + u < nk) {
#pragma unroll
        for (int mt = 0; mt < MT; mt++) {
          f16x8 av;
          if constexpr (NORM) {
#pragma unroll
            for (int j = 0; j < 4; j++) {
              const float x0 = ac[mt][u].lo[j], x1 = ac[mt][u].hi[j];
              ss[mt] += x0 * x0 + x1 * x1;
              av[j] = (f16_t)(x0 * gc[u][0][j]);
              av[4 + j] = (f16_t)(x1 * gc[u][1][j]);
            }
          } else {
            av = ac[mt][u].lo;
          }
#pragma unroll
          for (int c = 0; c < NC; c++) acc[mt][c] = __builtin_amdgcn_mfma_f32_16x16x32_f16(av, bc[c][u], acc[mt][c], 0, 0, 0);
        }
      }
    }
#pragma unroll
    for (int u = 0; u < U; u++) {
#pragma unroll
      for (int c = 0; c < NC; c++) bc[c][u] = bn[c][u];
      if constexpr (NORM) { gc[u][0] = gn[u][0]; gc[u][1] = gn[u][1]; }
#pragma unroll
      for (int mt = 0; mt < MT; mt++) ac[mt][u] = an[mt][u];
    }
  }
  // reduce the K-slices of the waves through LDS, in wave order
#pragma unroll
  for (int mt = 0; mt < MT; mt++) {
#pragma unroll
    for (int c = 0; c < NC; c++) red[wave][mt * NC + c][lane] = acc[mt][c];
    if constexpr (NORM) {
      float t = ss[mt];
      t += __shfl_xor(t, 16, 64);
      t += __shfl_xor(t, 32, 64);
      if ((lane >> 4) == 0) sq[wave][mt][lane & 15] = t;
    }
  }
  __syncthreads();
  for (int t = wave; t < MT * NC; t += NW) {
    const int mt = t / NC, ntc = nt * NC + t % NC;     // row tile and column tile of this result tile
    const int n = ntc * 16 + (lane & 15);
    f32x4 v = red[0][t][lane];
#pragma unroll
    for (int w = 1; w < NW; w++) v += red[w][t][lane];
    if constexpr (NORM) {
#pragma unroll
      for (int i = 0; i < 4; i++) {
        const int row = (lane >> 4) * 4 + i;
        float tot = sq[0][mt][row];
#pragma unroll
        for (int w = 1; w < NW; w++) tot += sq[w][mt][row];
        v[i] *= 1.0f / sqrtf(tot / (float)a.K + a.eps);
      }
    }
    if constexpr (EPI == EPI_QKV) {
      // tile nt of the fused projection: part 0/1/2 = q/k/v, head hh, and for q and k the rotary pairs
      // qd*8 .. +8 (columns 0..7 = first halves, 8..15 = second halves), for v the dims qd*16 .. +16
      const int d = a.H * FM_HD, col = lane & 15;
      const int part = (ntc * 16) / d, cp = (ntc * 16) % d;
      const int hh = cp >> 6, qd = (cp & 63) >> 4;
#pragma unroll
      for (int i = 0; i < 4; i++) {
        const long m = m0 + mt * 16 + (lane >> 4) * 4 + i;
        const long mc = m < a.M ? m : a.M - 1;
        float val = v[i];
        int dim;
        if (part < 2) {
          const int j = qd * 8 + (col & 7);
          const float2 t = a.cs[mc * 32 + j];
          const float o = __shfl_xor(val, 8, 64);
          val = col < 8 ? val * t.x - o * t.y : val * t.x + o * t.y;
          dim = col < 8 ? j : j + 32;
        } else {
          dim = qd * 16 + col;
        }
        if (m < a.M) {
          if (part == 0) {
            ((f16_t*)a.Y)[m * a.ldy + hh * FM_HD + dim] = (f16_t)val;
          } else {
            const int pa = a.pos[m];
            if (pa >= 0) {
              const int p = pa % (a.capb * 32);      // the cache is a ring when a window is set
              const long base = (m / a.RPS) * a.seq_stride + (long)hh * a.capb * 2048;
              if (part == 1) ((f16_t*)a.Kc)[base + kblk_off(p, dim)] = (f16_t)val;
              else ((f16_t*)a.Vc)[base + vblk_off(p, dim)] = (f16_t)val;
            }
          }
        }
      }
    } else if (n < a.N) {
#pragma unroll
      for (int i = 0; i < 4; i++) {
        const long m = m0 + mt * 16 + (lane >> 4) * 4 + i;
        if (m < a.M) {
          float val = v[i];
          if (EPI == EPI_F32) {
            if (a.R) val += a.R[(long)g * a.gsr + m * a.ldr + n];
            ((float*)a.Y)[(long)g * a.gsy + m * a.ldy + n] = val;
          } else {
            ((f16_t*)a.Y)[(long)g * a.gsy + m * a.ldy + n] = (f16_t)(EPI == EPI_GELU_T ? gelu_tanh_f(val) : val);
          }
        }
      }
    }
  }
}

struct MfmaRes {      // per-context resources of the MFMA kernels
  float* attn_ws;
  unsigned* attn_counters;
  size_t attn_ws_floats;
  int gemm_waves;     // 0 = choose per launch; 4, 8, 16 = forced (measurement switch)
  int gemm_mt_cap;    // 0 = default (below); 2, 3, 5, 8 = one workgroup covers up to that many 16-row tiles (measurement switch)
  int attn_wgs;       // key ranges of a growing cache: as few as give about this many workgroups per launch (768 by default,
                      // as for the condition memory); 0 = ranges as short as 8 blocks whatever the batch (measurement switch)
  int attn_merge;     // 2 = the last workgroup of a (sequence, head) always merges, publication without an L2 write-back (measurement)
  int gemm_nc;        // 0 = two column tiles per workgroup for the wide projections; 1 = one everywhere, 2 = two everywhere (measurement switches)
};

template <int MT, bool NORM, int NW, int NC>
void gemm_mfma_dispatch3(const GemmArgs& a, const GemmSplit& sp, int epi, dim3 grid, hipStream_t st) {
  if (epi == EPI_QKV) {
    if constexpr (NORM) hipLaunchKernelGGL((k_gemm_mfma<MT, EPI_QKV, true, NW, NC>), grid, dim3(NW * 64), 0, st, a, sp);
    return;
  }
  if (epi == EPI_F32) hipLaunchKernelGGL((k_gemm_mfma<MT, EPI_F32, NORM, NW, NC>), grid, dim3(NW * 64), 0, st, a, sp);
  else if (epi == EPI_GELU_T) hipLaunchKernelGGL((k_gemm_mfma<MT, EPI_GELU_T, NORM, NW, NC>), grid, dim3(NW * 64), 0, st, a, sp);
  else hipLaunchKernelGGL((k_gemm_mfma<MT, EPI_T, NORM, NW, NC>), grid, dim3(NW * 64), 0, st, a, sp);
}
template <int MT, bool NORM, int NC>
void gemm_mfma_dispatch2(const GemmArgs& a, const GemmSplit& sp, int nw, int epi, dim3 grid, hipStream_t st) {
  if constexpr (MT <= 3) { if (nw == 16) { gemm_mfma_dispatch3<MT, NORM, 16, NC>(a, sp, epi, grid, st); return; } }
  if constexpr (MT <= 5) { if (nw >= 8) { gemm_mfma_dispatch3<MT, NORM, 8, NC>(a, sp, epi, grid, st); return; } }
  gemm_mfma_dispatch3<MT, NORM, 4, NC>(a, sp, epi, grid, st);
}
template <int MT>
void gemm_mfma_dispatch(const GemmArgs& a, const GemmSplit& sp, int nw, int epi, int nc, dim3 grid, hipStream_t st) {
  if constexpr (MT == 1) {
    if (nc == 2) {
      if (a.gain) gemm_mfma_dispatch2<1, true, 2>(a, sp, nw, epi, grid, st);
      else gemm_mfma_dispatch2<1, false, 2>(a, sp, nw, epi, grid, st);
      return;
    }
  }
  if (a.gain) gemm_mfma_dispatch2<MT, true, 1>(a, sp, nw, epi, grid, st);
  else gemm_mfma_dispatch2<MT, false, 1>(a, sp, nw, epi, grid, st);
}

template <typename T>
bool mfma_gemm_launch(const MfmaRes&, const GemmArgs&, int, int, hipStream_t) { return false; }

template <>
inline bool mfma_gemm_launch<f16_t>(const MfmaRes& res, const GemmArgs& a, int epi, int groups, hipStream_t st) {
  if (a.K % 32 != 0 || a.M < 1) return false;
  const int KT = a.K / 32, Npad = (a.N + 15) / 16 * 16, NT = Npad / 16;
  const int mtiles = (a.M + 15) / 16;
  // Row tiles per workgroup.  Up to 128 rows (every launch of a decode step) a workgroup takes one 16-row tile and the
  // row tiles of a column tile go to different workgroups: the weight tile is then fetched once from HBM and again from
  // L2, but each workgroup reads a fifth of the activations at 72 rows and five times as many workgroups pull on the
  // weights (measured: -5 % per verify pass on 8 sequences at d = 1024, -7 % on 4 sequences at d = 1536).  Taller
  // problems (the per-block prefill GEMM) keep 128 rows per workgroup.
  int MT = mtiles <= 8 ? 1 : 8;
  if (res.gemm_mt_cap > 1) {
    MT = mtiles <= 1 ? 1 : mtiles <= 2 ? 2 : mtiles <= 3 ? 3 : mtiles <= 5 ? 5 : 8;
    if (MT > res.gemm_mt_cap) MT = res.gemm_mt_cap >= 8 ? 8 : res.gemm_mt_cap >= 5 ? 5 : res.gemm_mt_cap;
  }
  const int nmb = (a.M + MT * 16 - 1) / (MT * 16);
  // waves per workgroup: enough for about 2048 waves in the launch, at least two K fragments per wave, and the
  // partial tiles of all waves within the static LDS limit
  // two column tiles per workgroup for the wide projections (q,k,v, FFN up, output head) when rows are split 16 per
  // workgroup: FM_GEMM_NC=1 switches it off (measurement)
  const int nc = (MT == 1 && NT >= (res.gemm_nc == 2 ? 2 : 128) && NT % 2 == 0 && res.gemm_nc != 1) ? 2 : 1;   // gemm_nc == 2: every even launch (measurement)
  const long wgs = (long)(NT / nc) * groups * nmb;
  const int nw_max = MT <= 3 ? 16 : MT <= 5 ? 8 : 4;
  int nw = 4;
  while (nw < nw_max && wgs * nw < 2048 && KT / (nw * 2) >= 2) nw *= 2;
  if (res.gemm_waves == 4 || res.gemm_waves == 8 || res.gemm_waves == 16) nw = res.gemm_waves < nw_max ? res.gemm_waves : nw_max;
  GemmSplit sp{(KT + nw - 1) / nw};   // the waves of a workgroup split K
  dim3 grid(NT / nc, 1, groups * nmb);
  switch (MT) {
    case 1: gemm_mfma_dispatch<1>(a, sp, nw, epi, nc, grid, st); break;
    case 2: gemm_mfma_dispatch<2>(a, sp, nw, epi, nc, grid, st); break;
    case 3: gemm_mfma_dispatch<3>(a, sp, nw, epi, nc, grid, st); break;
    case 5: gemm_mfma_dispatch<5>(a, sp, nw, epi, nc, grid, st); break;
    default: gemm_mfma_dispatch<8>(a, sp, nw, epi, nc, grid, st); break;
  }
  return true;
}

