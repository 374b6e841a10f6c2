// Decode-path kernels (gfx950): the skinny GEMM and the block attention that every operator of a verify pass and of the draft
// heads is made of, in both storage types (T = half or float; what follows says "half" where the storage type is meant).
//
// A pass is a chain of several hundred dependent launches of 9 to ~100 rows each, so what bounds it is the length of one
// launch, not a rate: a launch boundary in a replayed graph costs 1.7 to 2.9 us on this chip, one trip to memory about
// 1 us.  The kernels here are therefore written for ONE trip to memory each: everything a workgroup will need (operand
// fragments, row statistics, residual, positions) is requested before the first value is used.
//
// Activations between launches ("tiled" buffers) are halves in MFMA operand order, [row tile of 16][K/32][64 lanes][8],
// like the weights: a fragment is one contiguous 1 KiB burst and goes from memory to the matrix core with no conversion.
// RMSNorm never reads a row twice: whoever produces the fp32 residual stream also stores half(x * gain) of the norm
// that comes next and, per 16 columns, the sum of squares of each row; the GEMM behind the norm adds those up and
// applies 1/rms, a scalar per row, to its result tile.
//
// Operands are swapped with respect to Y = X W^T (the weight fragment is operand A): a lane of the result tile then
// owns ONE row and four neighbouring columns, so that residual loads and all stores are vectors and the row scale is
// one value per lane.
#pragma once
#include <type_traits>
#include "fm_device.h"
#include "fm_kernels_mfma.h"

// element offset of (row m, column n) in a tiled buffer of KT = columns / 32
__device__ __forceinline__ long tile_off(int m, int n, int KT) {
  return ((long)(m >> 4) * KT + (n >> 5)) * 512 + ((m & 15) + 16 * ((n & 31) >> 3)) * 8 + (n & 7);
}

// Row r of a row set [sequence][row q of the sequence] -> (group, row of the group) of a grouped GEMM: `G` parameter
// sets, `mult` rows of a sequence per set, sets numbered from `base`, `tiles` row tiles per group.
struct RowMap {
  int G, mult, base, tiles;
};
__device__ __forceinline__ long map_off(const RowMap& rm, int s, int q, int n, int KT) {
  const int g = rm.G == 1 ? 0 : q % rm.G, k = rm.G == 1 ? q : q / rm.G;
  return (long)(rm.base + g) * rm.tiles * KT * 512 + tile_off(s * rm.mult + k, n, KT);
}

// ------------------------------------------------------------------------------------------
// GEMM
// ------------------------------------------------------------------------------------------
enum { DE_RES = 0, DE_GELU, DE_ROW, DE_TILE, DE_F32, DE_QKV, DE_ROPE };
// The norm in front of a GEMM: none; its input is x * gain already and comes with the row sums of squares; or the input is fp32 rows, scattered in
// memory, and every workgroup norms them, in fp32 as k_dec_rmsnorm does (the draft heads, whose rows no GEMM has left in operand order:
// a launch of 4 us less for each of their four norms).
enum { DN_NONE = 0, DN_SSQ, DN_ROWS };

struct DecGemm {
  const void* A; long gsa;       // tiled activations, elements per group
  const void* W; long gsw;       // tiled weights, elements per group
  int M, N, KT;                  // rows per group, columns, K / 32
  const float* ssq;              // DN_SSQ: [row tile][K/16][16] sums of squares of 16 columns each
  const float* const* src;       // DN_ROWS: fp32 rows by pointer, row m of a group at src[m * ldc + group]
  const float* sgain;            // and their gain, K values per group
  float inv_k, eps;              // inv_k: DN_SSQ
  const int* run_flag;           // the launch is skipped when *run_flag == 0 (may be null)
  // outputs (which of them: the epilogue)
  void* Y; long ldy, gsy;        // row-major output: fp32 (DE_RES, DE_F32) or half (DE_ROW, DE_QKV q, DE_ROPE)
  const float* R; long ldr;      // fp32 rows added (DE_RES; may be null, may be Y)
  const float* const* Rt;        // DE_F32: fp32 rows added, by pointer as src (may be null)
  void* X; long gsx;             // tiled half output of width N (DE_GELU, DE_TILE; DE_RES: x * gain, may be null)
  const float* gain;             // DE_RES: gain of the norm that follows
  float* ssq_out;                // DE_RES: [row tile][N/16][16]
  const int* pos;                // DE_RES with rings, DE_QKV: position of each row, -1 = inactive
  int RPS;                       // rows per sequence
  float *tap, *ring; int rs;     // DE_RES: rings (rs entries per sequence) that receive the old row (tap) and the new row
  const float2* cs;              // DE_QKV, DE_ROPE: [row][hd/2] (cos, sin); DE_ROPE: row = m * ldc + group
  int ldc, hd;                   // rows of a table (cs, src, Rt) between two rows of a group
  void *Kc, *Vc; long seq_stride; int capb, H;   // DE_QKV: blocked caches
};

// MT row tiles x NC column tiles of 16 per workgroup, NW waves split K.
// U fragments per wave and chunk: the first chunk (all of the K slice for the usual shapes) is in flight before
// anything is waited for, later chunks one ahead.
template <typename T, int MT, int NC, int NW, int U, bool LOOP, int EPI, int NORM>
__global__ __launch_bounds__(NW * 64) void k_dec_gemm(DecGemm a) {
  typedef typename Op<T>::V8 V8;
  typedef typename Op<T>::V4 V4;
  constexpr int NTILE = MT * NC;
  extern __shared__ f32x4 dg_smem[];
  f32x4* red = dg_smem;                                    // [NW][tiles][64]
  float* sq = (float*)(dg_smem + NW * NTILE * 64);             // [NW][MT][16]
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int g = lane >> 4, rl = lane & 15;
  const int grp = blockIdx.z, mb = blockIdx.y, nt0 = blockIdx.x * NC;
  const int rf = a.run_flag ? *a.run_flag : 1;
  const int KT = a.KT, mt0 = mb * MT;
  const int ntile = (a.M + 15) / 16;
  const T* Ap = (const T*)a.A + (long)grp * a.gsa + lane * 8;
  const T* Wp = (const T*)a.W + (long)grp * a.gsw + (long)nt0 * KT * 512 + lane * 8;
  const int FW = (KT + NW - 1) / NW, kt0 = wave * FW, nk = min(FW, KT - kt0);
  f32x4 acc[MT][NC];
#pragma unroll
  for (int mt = 0; mt < MT; mt++)
#pragma unroll
    for (int c = 0; c < NC; c++) acc[mt][c] = f32x4{0.f, 0.f, 0.f, 0.f};
  V8 wc[NC][U], ac[MT][U];
  // rows by pointer: the pointers are asked for first, so that waiting for them waits for nothing else
  const float *xrow = nullptr, *rrow = nullptr;
  if constexpr (NORM == DN_ROWS) xrow = a.src[(long)min(mt0 * 16 + rl, a.M - 1) * a.ldc + grp];
  if (EPI == DE_F32 && a.Rt && wave < NTILE) rrow = a.Rt[(long)min((mt0 + wave / NC) * 16 + rl, a.M - 1) * a.ldc + grp];
  auto load_chunk = [&](V8 (&w)[NC][U], V8 (&x)[MT][U], int i0) {
#pragma unroll
    for (int u = 0; u < U; u++)
      if (i0 + u < nk) {
        const long kt = kt0 + i0 + u;
#pragma unroll
        for (int c = 0; c < NC; c++) w[c][u] = *reinterpret_cast<const V8*>(Wp + ((long)c * KT + kt) * 512);
#pragma unroll
        for (int mt = 0; mt < (NORM == DN_ROWS ? 0 : MT); mt++) {
          const int t = min(mt0 + mt, ntile - 1);          // a tile past the last one is computed on the last one's rows, never stored
          x[mt][u] = *reinterpret_cast<const V8*>(Ap + ((long)t * KT + kt) * 512);
        }
      }
  };
  load_chunk(wc, ac, 0);
  float ss[MT];
  f32x4 xv[NORM == DN_ROWS ? U : 1][2], gn[NORM == DN_ROWS ? U : 1][2];
  if constexpr (NORM == DN_ROWS) {
    static_assert(MT == 1 && !LOOP);
    const float* gp = a.sgain + (long)grp * KT * 32;
#pragma unroll
    for (int u = 0; u < U; u++)
      if (u < nk) {
        const int k = (kt0 + u) * 32 + g * 8;
#pragma unroll
        for (int h = 0; h < 2; h++) { gn[u][h] = *reinterpret_cast<const f32x4*>(gp + k + 4 * h); xv[u][h] = *reinterpret_cast<const f32x4*>(xrow + k + 4 * h); }
      }
  }
  // operands of the epilogue of this wave's first result tile
  const int tm = wave / NC, tc = wave % NC;
  const int em = (mt0 + tm) * 16 + rl, en = (nt0 + tc) * 16 + g * 4;
  const bool eon = wave < NTILE && em < a.M;
  f32x4 rv = f32x4{0.f, 0.f, 0.f, 0.f}, gv = rv, c0 = rv, c1 = rv;
  int ep = -1;
  if (eon) {
    if (EPI == DE_RES && a.R) rv = *reinterpret_cast<const f32x4*>(a.R + (long)em * a.ldr + en);
    if (EPI == DE_F32 && a.Rt && a.N % 16 == 0) rv = *reinterpret_cast<const f32x4*>(rrow + en);
    if (EPI == DE_RES) {
      if (a.gain) gv = *reinterpret_cast<const f32x4*>(a.gain + en);
      if (a.pos) ep = a.pos[em];
    }
    if (EPI == DE_QKV || EPI == DE_ROPE) {
      if (EPI == DE_QKV) ep = a.pos[em];
      const int part = EPI == DE_QKV ? ((nt0 + tc) * 16) / (a.H * a.hd) : 0;
      if (part < 2) {
        const int qd = ((nt0 + tc) % (a.hd >> 4));
        const long row = EPI == DE_QKV ? em : (long)em * a.ldc + grp;
        const f32x4* cp = reinterpret_cast<const f32x4*>(a.cs + row * (a.hd >> 1) + qd * 8 + (g & 1) * 4);
        c0 = cp[0]; c1 = cp[1];
      }
    }
  }
  if constexpr (NORM == DN_SSQ) {
    const int ns = KT * 2;
#pragma unroll
    for (int mt = 0; mt < MT; mt++) {
      const float* sp = a.ssq + (long)min(mt0 + mt, ntile - 1) * ns * 16 + rl;
      float t = 0.f;
      for (int i = wave * 4 + g; i < ns; i += NW * 4) t += sp[i * 16];
      ss[mt] = t;
    }
  }
  asm volatile("" ::: "memory");      // the loads above stay above the exit
  if (rf == 0) return;
  if constexpr (NORM == DN_ROWS) {
    // The row factor comes before the rounding to half: a row may be far from 1 (the residual stream grows, a head's linear layer has any scale), and
    // x * gain alone would leave the range of half or lose bits to its subnormals.
    float t = 0.f;
#pragma unroll
    for (int u = 0; u < U; u++)
      if (u < nk)
#pragma unroll
        for (int j = 0; j < 8; j++) t += xv[u][j >> 2][j & 3] * xv[u][j >> 2][j & 3];
    t = rows_sum(t);
    if (g == 0) sq[wave * 16 + rl] = t;
    __syncthreads();
    float tot = sq[rl];
#pragma unroll
    for (int w = 1; w < NW; w++) tot += sq[w * 16 + rl];
    const float inv = 1.0f / sqrtf(tot / (float)(KT * 32) + a.eps);
#pragma unroll
    for (int u = 0; u < U; u++)
      if (u < nk)
#pragma unroll
        for (int j = 0; j < 8; j++) ac[0][u][j] = (T)(xv[u][j >> 2][j & 3] * inv * gn[u][j >> 2][j & 3]);
  }
  auto mul_chunk = [&](V8 (&w)[NC][U], V8 (&x)[MT][U], int i0) {
#pragma unroll
    for (int u = 0; u < U; u++)
      if (i0 + u < nk) {
#pragma unroll
        for (int mt = 0; mt < MT; mt++)
#pragma unroll
          for (int c = 0; c < NC; c++) acc[mt][c] = Op<T>::mul(w[c][u], x[mt][u], acc[mt][c]);
      }
  };
  if constexpr (LOOP) {
    for (int i0 = 0; i0 < nk; i0 += 2 * U) {
      V8 wn[NC][U], an[MT][U];
      load_chunk(wn, an, i0 + U);
      mul_chunk(wc, ac, i0);
      load_chunk(wc, ac, i0 + 2 * U);
      mul_chunk(wn, an, i0 + U);
    }
  } else {
    mul_chunk(wc, ac, 0);
  }
  // the waves' K slices meet in LDS and are added in wave order
#pragma unroll
  for (int mt = 0; mt < MT; mt++) {
#pragma unroll
    for (int c = 0; c < NC; c++) red[(wave * NTILE + mt * NC + c) * 64 + lane] = acc[mt][c];
    if constexpr (NORM == DN_SSQ) {
      const float t = rows_sum(ss[mt]);
      if (g == 0) sq[(wave * MT + mt) * 16 + rl] = t;
    }
  }
  __syncthreads();
  for (int t = wave; t < NTILE; t += NW) {
    const int mt = t / NC, ntc = nt0 + t % NC;
    const int m = (mt0 + mt) * 16 + rl, n = ntc * 16 + g * 4;
    f32x4 v = red[t * 64 + lane];
#pragma unroll
    for (int w = 1; w < NW; w++) v += red[(w * NTILE + t) * 64 + lane];
    if constexpr (NORM == DN_SSQ) {
      float tot = sq[mt * 16 + rl];
#pragma unroll
      for (int w = 1; w < NW; w++) tot += sq[(w * MT + mt) * 16 + rl];
      v *= 1.0f / sqrtf(tot * a.inv_k + a.eps);
    }
    const bool on = m < a.M;
    const bool first = t == wave && NTILE <= NW;     // operands already here
    if constexpr (EPI == DE_RES) {
      if (on) {
        if (!first && a.R) rv = *reinterpret_cast<const f32x4*>(a.R + (long)m * a.ldr + n);
        if (!first && a.gain) gv = *reinterpret_cast<const f32x4*>(a.gain + n);
        if (!first && a.pos) ep = a.pos[m];
        v += rv;
        *reinterpret_cast<f32x4*>((float*)a.Y + (long)m * a.ldy + n) = v;
        if (a.X) {
          V4 o;
#pragma unroll
          for (int i = 0; i < 4; i++) o[i] = (T)(v[i] * gv[i]);
          *reinterpret_cast<V4*>((T*)a.X + tile_off(m, n, a.N >> 5)) = o;
        }
        if (ep >= 0) {
          const long ro = ((long)(m / a.RPS) * a.rs + (ep & (a.rs - 1))) * a.N + n;
          if (a.tap) *reinterpret_cast<f32x4*>(a.tap + ro) = rv;
          if (a.ring) *reinterpret_cast<f32x4*>(a.ring + ro) = v;
        }
      }
      if (a.ssq_out) {
        const float s2 = rows_sum(v[0] * v[0] + v[1] * v[1] + v[2] * v[2] + v[3] * v[3]);
        if (g == 0 && on) a.ssq_out[((long)(mt0 + mt) * (a.N >> 4) + ntc) * 16 + rl] = s2;
      }
    } else if constexpr (EPI == DE_GELU || EPI == DE_TILE) {
      if (on) {
        V4 o;
#pragma unroll
        for (int i = 0; i < 4; i++) o[i] = (T)(EPI == DE_GELU ? gelu_tanh_f(v[i]) : v[i]);
        *reinterpret_cast<V4*>((T*)a.X + (long)grp * a.gsx + tile_off(m, n, a.N >> 5)) = o;
      }
    } else if constexpr (EPI == DE_ROW) {
      if (on) {
        V4 o;
#pragma unroll
        for (int i = 0; i < 4; i++) o[i] = (T)v[i];
        *reinterpret_cast<V4*>((T*)a.Y + (long)grp * a.gsy + (long)m * a.ldy + n) = o;
      }
    } else if constexpr (EPI == DE_F32) {
      if (on) {
        float* y = (float*)a.Y + (long)grp * a.gsy + (long)m * a.ldy + n;
        if (a.N % 16 == 0) {
          if (!first && a.Rt) rv = *reinterpret_cast<const f32x4*>(a.Rt[(long)m * a.ldc + grp] + n);
          v += rv;
          *reinterpret_cast<f32x4*>(y) = v;
        } else {
#pragma unroll
          for (int i = 0; i < 4; i++)
            if (n + i < a.N) y[i] = v[i] + (a.Rt ? a.Rt[(long)m * a.ldc + grp][n + i] : 0.f);
        }
      }
    } else {
      // q, k, v projection (or the q projection of the draft heads).  Tiles of the q and k parts hold 8 rotary pairs of a
      // head: columns 0..7 the first halves, 8..15 the second halves, so the partner of a value sits 32 lanes away.
      const int d = a.H * a.hd, part = EPI == DE_QKV ? (ntc * 16) / d : 0, cp = ntc * 16 - part * d;
      const int hh = cp / a.hd, qd = (cp - hh * a.hd) >> 4;
      int dim = qd * 16 + g * 4;
      if (part < 2) {
        if (!first) {
          const long row = EPI == DE_QKV ? min(m, a.M - 1) : (long)min(m, a.M - 1) * a.ldc + grp;
          const f32x4* cq = reinterpret_cast<const f32x4*>(a.cs + row * (a.hd >> 1) + qd * 8 + (g & 1) * 4);
          c0 = cq[0]; c1 = cq[1];
        }
        const f32x4 cx = {c0[0], c0[2], c1[0], c1[2]}, sx = {c0[1], c0[3], c1[1], c1[3]};
#pragma unroll
        for (int i = 0; i < 4; i++) {
          const float o = lane_xor32(v[i]);
          v[i] = g < 2 ? v[i] * cx[i] - o * sx[i] : v[i] * cx[i] + o * sx[i];
        }
        dim = (g < 2 ? 0 : a.hd >> 1) + qd * 8 + (g & 1) * 4;
      }
      if (on) {
        V4 o;
#pragma unroll
        for (int i = 0; i < 4; i++) o[i] = (T)v[i];
        if (part == 0) {
          *reinterpret_cast<V4*>((T*)a.Y + (long)grp * a.gsy + (long)m * a.ldy + hh * a.hd + dim) = o;
        } else {
          if (!first) ep = a.pos[m];
          if (ep >= 0) {
            const int p = ep % (a.capb * 32);        // the cache is a ring when a window is set
            const int r = p & 31;
            const long base = (long)(m / a.RPS) * a.seq_stride + ((long)hh * a.capb + (p >> 5)) * (32 * a.hd);
            if (part == 1) {
              const int f = (r >> 4) * (a.hd >> 5) + (dim >> 5), ln = (r & 15) + 16 * ((dim & 31) >> 3);
              *reinterpret_cast<V4*>((T*)a.Kc + base + (f * 64 + ln) * 8 + (dim & 7)) = o;
            } else {
              const int slot = ((r & 15) >> 2) * 8 + (r >> 4) * 4 + (r & 3);
#pragma unroll
              for (int i = 0; i < 4; i++) ((T*)a.Vc)[base + (dim + i) * 32 + slot] = o[i];
            }
          }
        }
      }
    }
  }
}

// ------------------------------------------------------------------------------------------
// Attention over a blocked K/V cache (layouts: kblk_off / vblk_off), up to 32 query rows of a sequence per workgroup
// ------------------------------------------------------------------------------------------
// The 32-key blocks of a head are dealt to the NW waves of `ns` workgroups in turn: block b belongs to wave b % NW of
// split (b / NW) % ns.  The deal depends on nothing but the launch configuration, so the arithmetic of one query row never
// depends on what else is in the block or on how far the sequence has grown (speculative and one-token decoding agree
// bit for bit), and it is balanced at every length: short contexts keep all keys in one workgroup (no merge), long
// ones use all of them.  Partial results of several splits are merged, in split order, by the workgroup that arrives last.
struct AttnSet {
  const void* q;             // [sequence][RS rows][d] rotated queries
  const int* limit;          // [sequence][RS] last visible key, -1 = inactive row
  int rows, q0, RS;          // this launch takes rows q0 .. q0 + rows of every sequence
  const void *Kc, *Vc;
  long seq_stride;           // elements between the caches of two sequences
  int capb, window, ns;      // capacity in blocks, sliding window (0 = none; the cache is then a ring), splits
  RowMap rm;                 // where the rows go in the tiled output
  void* out;
};
#define FM_ATTN_SETS 4
// Weights that a launch reads ahead for the ones behind it: `groups` column tiles of `bytes` each.
struct WeightRange { const void* W; int bytes, groups; };
struct AttnArgs {
  AttnSet set[FM_ATTN_SETS];     // first member of the only kernel argument (attn_set)
  int S, H, ns_max;
  unsigned* arrived;         // [set][sequence][head] splits that have published their part, zero between launches
  float* ws;                 // [set][sequence][head][ns_max][QT*16*HD unnormalised O | QT*16 running max (log2 units) | QT*16 sums]
  const int* run_flag;
  int nset, ahead;           // planes of the grid (blockIdx.z) that attend: nset * S; `ahead` more read weights ahead
  WeightRange next[4];
};
// the set of this workgroup, read from the argument segment itself: indexing the by-value argument would copy it to scratch memory
typedef const __attribute__((address_space(4))) AttnSet* attn_set_t;
__device__ __forceinline__ attn_set_t attn_set(int z) {
  return (attn_set_t)((const __attribute__((address_space(4))) char*)__builtin_amdgcn_kernarg_segment_ptr() + (size_t)z * sizeof(AttnSet));
}
__device__ __forceinline__ int attn_active(int maxlim, int capb, int ns, int NW) {      // splits that hold visible keys
  const int nblk = min((maxlim + 32) >> 5, capb);
  return max(1, min(ns, (nblk + NW - 1) / NW));
}

// ONCE: keys and values as non-temporal loads (attn_once)
template <typename T, int QT, int HD, int NW, bool ONCE>
__global__ __launch_bounds__(NW * 64) void k_dec_attn(AttnArgs a) {
  typedef typename Op<T>::V8 V8;
  typedef typename Op<T>::V4 V4;
  constexpr int NQ = QT * 16, KC = HD / 32, DT = HD / 16, BLK = 32 * HD, PSZ = NQ * HD + 2 * NQ, LD = HD + 4;
  extern __shared__ f32x4 da_smem[];
  float* lo = (float*)da_smem;              // [NW][NQ][LD]
  float* lm = lo + NW * NQ * LD;            // [NW][NQ]
  float* ll = lm + NW * NQ;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int g = lane >> 4, ql = lane & 15;
  const int hh = blockIdx.x, split = blockIdx.y, s = blockIdx.z % a.S, z = blockIdx.z / a.S;
  if (z >= a.nset) {
    // Read ahead: the GEMMs behind this launch wait for cold weights, about a third of their 4 us, while a short attention leaves the
    // memory and compute units idle.  L2 outlives a launch; each die has its own, and workgroup i runs on die i mod 8, as do the column tiles
    // i mod 8 of a GEMM (only the speed depends on that).  The data goes to LDS and is never looked at.
    if (a.run_flag && *a.run_flag == 0) return;
    const int plane = gridDim.x * gridDim.y, base = plane * a.nset * a.S, id = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
    const int die = id & 7, rank = (id - base) >> 3, ranks = max(1, (plane * a.ahead) >> 3);
    if (rank >= ranks) return;
#pragma unroll
    for (int r = 0; r < 4; r++) {
      const int bytes = a.next[r].bytes, groups = a.next[r].groups;
      for (int x = die + 8 * rank; x < groups; x += 8 * ranks) {
        const char* src = (const char*)a.next[r].W + (long)x * bytes + lane * 16;
        for (int o = wave * 1024; o < bytes; o += NW * 1024)
          __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src + o),
                                           (__attribute__((address_space(3))) void*)((char*)da_smem + wave * 1024), 16, 0, 0);
      }
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);          // vmcnt(0)
    return;
  }
  const attn_set_t A = attn_set(z);
  const RowMap rm{A->rm.G, A->rm.mult, A->rm.base, A->rm.tiles};
  if (split >= A->ns) return;
  const int rf = a.run_flag ? *a.run_flag : 1;
  const int d = a.H * HD;
  const float kScale = (HD == 64 ? 0.125f : 1.0f / sqrtf((float)HD)) * 1.4426950408889634f;   // 1/sqrt(HD) * log2(e)
  const T* Kb = (const T*)A->Kc + (long)s * A->seq_stride + (long)hh * A->capb * BLK + lane * 8;
  const T* Vb = (const T*)A->Vc + (long)s * A->seq_stride + (long)hh * A->capb * BLK + ql * 32 + g * 8;
  // the first block of this wave is inside the cache whatever the length: request it before anything else is known
  const int bstep = A->ns * NW;
  int b = split * NW + wave;
  V8 kf[2 * KC], vf[DT];
  auto fetch = [](const V8* p) { return ONCE ? __builtin_nontemporal_load(p) : *p; };
  auto load_k = [&](int blk) {
#pragma unroll
    for (int f = 0; f < 2 * KC; f++) kf[f] = fetch(reinterpret_cast<const V8*>(Kb + (long)blk * BLK + f * 512));
  };
  auto load_v = [&](int blk) {
#pragma unroll
    for (int dt = 0; dt < DT; dt++) vf[dt] = fetch(reinterpret_cast<const V8*>(Vb + (long)blk * BLK + dt * 512));
  };
  load_k(min(b, A->capb - 1));
  load_v(min(b, A->capb - 1));
  int lim[QT], first[QT];
  V8 qf[QT][KC];
  int maxlim = -1;
#pragma unroll
  for (int t = 0; t < QT; t++) {
    const int qi = t * 16 + ql;
    const bool on = qi < A->rows;
    const long row = (long)s * A->RS + A->q0 + (on ? qi : 0);
    lim[t] = on ? A->limit[row] : -1;
    const T* qp = (const T*)A->q + row * d + hh * HD + g * 8;
#pragma unroll
    for (int kc = 0; kc < KC; kc++) qf[t][kc] = *reinterpret_cast<const V8*>(qp + kc * 32);
  }
  asm volatile("" ::: "memory");      // the loads above stay above the exit
  if (rf == 0) return;
#pragma unroll
  for (int t = 0; t < QT; t++) {
    first[t] = A->window > 0 ? max(lim[t] - A->window + 1, 0) : 0;     // sliding window: keys first .. lim
    maxlim = max(maxlim, lim[t]);
  }
  maxlim = __builtin_amdgcn_readfirstlane(row16_max(maxlim));
  // With a window the cache is a ring of capb blocks: position p lives in slot p mod (32 capb), and a slot holds
  // the latest position written to it.  Seen from the newest visible position `maxlim`, slot j holds lapbase + j if that
  // is <= maxlim, else the position one lap earlier (anything newer in the ring is a stale row of a rejected block: it
  // maps below the window and is masked).  Without a window lapbase = 0.
  const int nblk = min((maxlim + 32) >> 5, A->capb);
  const int ringn = A->capb * 32;
  const int lapbase = A->window > 0 ? max(maxlim, 0) / ringn * ringn : 0;
  const int nact = attn_active(maxlim, A->capb, A->ns, NW);
  if (split >= nact) return;

  float mrun[QT], lrun[QT];
  f32x4 o[QT][DT];
#pragma unroll
  for (int t = 0; t < QT; t++) {
    mrun[t] = -INFINITY;
    lrun[t] = 0.f;
#pragma unroll
    for (int dt = 0; dt < DT; dt++) o[t][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  // The operands of the next block are requested into the registers of this one as soon as those are free: its keys behind the
  // score products, its values behind the output products.
  for (; b < nblk; b += bstep) {
    const int bn = min(b + bstep, A->capb - 1);
    // scores, transposed: sT[t][hb][i] = <K[key], Q[q]> for key = b*32 + hb*16 + g*4 + i, q = this lane's row
    f32x4 sT[QT][2];
#pragma unroll
    for (int t = 0; t < QT; t++)
#pragma unroll
      for (int hb = 0; hb < 2; hb++) {
        f32x4 zz = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int kc = 0; kc < KC; kc++) zz = Op<T>::mul(kf[hb * KC + kc], qf[t][kc], zz);
        sT[t][hb] = zz;
      }
    if (b + bstep < nblk) load_k(bn);
#pragma unroll
    for (int t = 0; t < QT; t++) {
      float mx = -INFINITY;
#pragma unroll
      for (int hb = 0; hb < 2; hb++)
#pragma unroll
        for (int i = 0; i < 4; i++) {
          int key = lapbase + b * 32 + hb * 16 + g * 4 + i;     // absolute position held by this slot
          key = key > maxlim ? key - ringn : key;
          const float v = (key <= lim[t] && key >= first[t]) ? sT[t][hb][i] * kScale : -INFINITY;
          sT[t][hb][i] = v;
          mx = fmaxf(mx, v);
        }
      mx = rows_max(mx);
      const float mnew = fmaxf(mrun[t], mx);
      const float msafe = mnew == -INFINITY ? 0.f : mnew;
      const float alpha = __builtin_amdgcn_exp2f(mrun[t] - msafe);   // exp2(-inf) = 0 on the first block
      mrun[t] = mnew;
      V8 pf;
      float psum = 0.f;
#pragma unroll
      for (int hb = 0; hb < 2; hb++)
#pragma unroll
        for (int i = 0; i < 4; i++) {
          const float p = __builtin_amdgcn_exp2f(sT[t][hb][i] - msafe);
          psum += p;
          pf[hb * 4 + i] = (T)p;
        }
      lrun[t] = lrun[t] * alpha + psum;
      // Slots that this stream has not reached hold what an earlier mesh left there.  Their probability is 0, but 0 times a value that is
      // not finite is NaN: they count as zero rows.  (Here, where the values are needed: in front of the scores it is 60 ns a launch.)
      if (t == 0 && lapbase == 0 && b * 32 + 31 > maxlim) {
#pragma unroll
        for (int dt = 0; dt < DT; dt++)
#pragma unroll
          for (int j = 0; j < 8; j++) vf[dt][j] = b * 32 + (j >> 2) * 16 + g * 4 + (j & 3) > maxlim ? (T)0.f : vf[dt][j];
      }
#pragma unroll
      for (int dt = 0; dt < DT; dt++) {
        o[t][dt] *= alpha;
        o[t][dt] = Op<T>::mul(vf[dt], pf, o[t][dt]);   // O^T[dim][q]
      }
    }
    if (b + bstep < nblk) load_v(bn);
  }
  // Combine the waves of the workgroup that had keys.  An inactive row carries a negative sum and gives 0; a row with keys whose
  // sum is NaN or 0 (scores that are not finite) gives NaN, which the pass counts.
#pragma unroll
  for (int t = 0; t < QT; t++) {
    const float l = rows_sum(lrun[t]);
    if (g == 0) { lm[wave * NQ + t * 16 + ql] = lim[t] < 0 ? 0.f : mrun[t]; ll[wave * NQ + t * 16 + ql] = lim[t] < 0 ? -1.f : l; }
#pragma unroll
    for (int dt = 0; dt < DT; dt++) *reinterpret_cast<f32x4*>(lo + (wave * NQ + t * 16 + ql) * LD + dt * 16 + g * 4) = o[t][dt];
  }
  __syncthreads();
  const int wact = max(1, min(NW, nblk - split * NW));
  float* part = a.ws + (((long)blockIdx.z * a.H + hh) * a.ns_max + split) * PSZ;
  for (int e = threadIdx.x; e < A->rows * (HD / 4); e += NW * 64) {
    const int qi = e / (HD / 4), dim = e % (HD / 4) * 4;
    float M = -INFINITY;
    for (int w = 0; w < wact; w++) M = fmaxf(M, lm[w * NQ + qi]);
    const float Ms = M == -INFINITY ? 0.f : M;
    f32x4 num = f32x4{0.f, 0.f, 0.f, 0.f};
    float den = 0.f;
    for (int w = 0; w < wact; w++) {
      const float f = __builtin_amdgcn_exp2f(lm[w * NQ + qi] - Ms);
      num += *reinterpret_cast<const f32x4*>(lo + (w * NQ + qi) * LD + dim) * f;
      den += ll[w * NQ + qi] * f;
    }
    if (nact == 1) {
      V4 ov;
#pragma unroll
      for (int i = 0; i < 4; i++) ov[i] = (T)(den < 0.f ? 0.f : num[i] / den);
      *reinterpret_cast<V4*>((T*)A->out + map_off(rm, s, A->q0 + qi, hh * HD + dim, d >> 5)) = ov;
    } else {
#pragma unroll
      for (int i = 0; i < 4; i++) st_agent(part + qi * HD + dim + i, num[i]);
      if (dim == 0) { st_agent(part + NQ * HD + qi, M); st_agent(part + NQ * HD + NQ + qi, den); }
    }
  }
  if (nact == 1) return;
  // The parts went out as agent-scope stores, written through to where all dies see them: once a wave's stores have completed
  // (vmcnt 0) they are visible, and no cache has to be written back.  The last of the active splits reads them all the same way.
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
  __builtin_amdgcn_s_waitcnt(0x0F70);          // vmcnt(0)
  __syncthreads();
  int* last = (int*)da_smem;
  if (threadIdx.x == 0) {
    unsigned* cnt = a.arrived + (long)blockIdx.z * a.H + hh;
    const unsigned old = __hip_atomic_fetch_add(cnt, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    *last = old == (unsigned)nact - 1;
    if (*last) __hip_atomic_store(cnt, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
  __syncthreads();
  if (!*last) return;
  const agent_buf_t parts = agent_buf(a.ws + ((long)blockIdx.z * a.H + hh) * a.ns_max * PSZ, nact * PSZ * 4);
  agent_again();
  constexpr int C = 8;      // splits whose parts a thread has in flight together
  for (int e = threadIdx.x; e < A->rows * (HD / 4); e += NW * 64) {
    const int qi = e / (HD / 4), dim = e % (HD / 4) * 4;
    float M = -INFINITY, den = 0.f;
    f32x4 num = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int k0 = 0; k0 < nact; k0 += C) {
      f32x4 v[C];
      float m[C], l[C];
#pragma unroll
      for (int j = 0; j < C; j++) {
        const int p = min(k0 + j, nact - 1) * PSZ;
        v[j] = __builtin_bit_cast(f32x4, ld_agent4(parts, (p + qi * HD + dim) * 4));
        m[j] = __uint_as_float(ld_agent1(parts, (p + NQ * HD + qi) * 4));
        l[j] = __uint_as_float(ld_agent1(parts, (p + NQ * HD + NQ + qi) * 4));
      }
      agent_again();      // all of them go out here: the compiler would move some behind the tests below, a second trip
      float Mc = M;
#pragma unroll
      for (int j = 0; j < C; j++)
        if (k0 + j < nact) Mc = fmaxf(Mc, m[j]);
      const float Ms = Mc == -INFINITY ? 0.f : Mc;
      const float sc = __builtin_amdgcn_exp2f(M - Ms);
      num *= sc;
      den *= sc;
      M = Mc;
#pragma unroll
      for (int j = 0; j < C; j++)
        if (k0 + j < nact) {
          const float f = __builtin_amdgcn_exp2f(m[j] - Ms);
          num += v[j] * f;
          den += l[j] * f;
        }
    }
    V4 ov;
#pragma unroll
    for (int i = 0; i < 4; i++) ov[i] = (T)(den < 0.f ? 0.f : num[i] / den);
    *reinterpret_cast<V4*>((T*)A->out + map_off(rm, s, A->q0 + qi, hh * HD + dim, d >> 5)) = ov;
  }
}

// ------------------------------------------------------------------------------------------
// Rows that enter the chain: normalised rows of the draft heads, pooled groups, upsampled rows
// ------------------------------------------------------------------------------------------
// sum of squares of 16 columns from the four lanes that hold four columns each
__device__ __forceinline__ float quad_sum(float v) {
  v += __shfl_xor(v, 1, 64);
  v += __shfl_xor(v, 2, 64);
  return v;
}
// four columns n.. of row m of a residual stream: fp32 row, half(x * gain) in tiled order, sum of squares per 16 columns
template <typename T>
__device__ __forceinline__ void put_row4(const f32x4& v, int m, int n, int d, float* h, T* xg, const float* gain, float* ssq) {
  *reinterpret_cast<f32x4*>(h + (long)m * d + n) = v;
  const f32x4 gv = *reinterpret_cast<const f32x4*>(gain + n);
  typedef typename Op<T>::V4 V4;
  V4 o;
#pragma unroll
  for (int i = 0; i < 4; i++) o[i] = (T)(v[i] * gv[i]);
  *reinterpret_cast<V4*>(xg + tile_off(m, n, d >> 5)) = o;
  const float t = quad_sum(v[0] * v[0] + v[1] * v[1] + v[2] * v[2] + v[3] * v[3]);
  if ((threadIdx.x & 3) == 0) ssq[((long)(m >> 4) * (d >> 4) + (n >> 4)) * 16 + (m & 15)] = t;
}

// RMSNorm of gathered rows into the tiled input of a grouped GEMM (row r = s * per_seq + q, gain of head r % gain_mod), where the GEMM does not
// take the rows itself (dec_gemm_rows)
template <typename T>
__global__ __launch_bounds__(256) void k_dec_rmsnorm(const float* const* __restrict__ srcptr, const float* __restrict__ gain, int gain_mod,
                                                      T* __restrict__ out, RowMap rm, int per_seq, int d,
                                                      float eps, const int* run_flag) {
  const int r = blockIdx.x;
  const int rf = run_flag ? *run_flag : 1;
  const float* x = srcptr[r];
  const float* g = gain + (long)(gain_mod ? r % gain_mod : 0) * d;
  __shared__ float red[4];
  if (rf == 0) return;
  float ss = 0.f;
  f32x4 v0 = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int n = threadIdx.x * 4; n < d; n += 1024) {
    const f32x4 v = *reinterpret_cast<const f32x4*>(x + n);
    if (n < 1024) v0 = v;
    ss += v[0] * v[0] + v[1] * v[1] + v[2] * v[2] + v[3] * v[3];
  }
  ss = wave_sum(ss);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = ss;
  __syncthreads();
  ss = red[0] + red[1] + red[2] + red[3];
  const float inv = 1.0f / sqrtf(ss / (float)d + eps);
  for (int n = threadIdx.x * 4; n < d; n += 1024) {
    const f32x4 v = n < 1024 ? v0 : *reinterpret_cast<const f32x4*>(x + n);
    const f32x4 gv = *reinterpret_cast<const f32x4*>(g + n);
    typename Op<T>::V4 o;
#pragma unroll
    for (int i = 0; i < 4; i++) o[i] = (T)(v[i] * inv * gv[i]);
    *reinterpret_cast<typename Op<T>::V4*>(out + map_off(rm, r / per_seq, r % per_seq, n, d >> 5)) = o;
  }
}

// coarse slot j pools fine rows 3j-2, 3j-1, 3j (rows before the start count as zero; always / 3)
template <typename T>
__global__ __launch_bounds__(256) void k_dec_pool3(const float* __restrict__ ring_fine, int RSf, const int* __restrict__ pos_coarse,
                                                    int RPS, T* __restrict__ out, int d, const int* run_flag) {
  const int r = blockIdx.x, j = pos_coarse[r], s = r / RPS;
  if (*run_flag == 0) return;
  for (int n = threadIdx.x * 4; n < d; n += 1024) {
    f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
    if (j >= 0) {
      for (int k = 3 * j - 2; k <= 3 * j; k++)
        if (k >= 0) acc += *reinterpret_cast<const f32x4*>(ring_fine + ((long)s * RSf + (k & (RSf - 1))) * d + n);
    }
    typename Op<T>::V4 o;
#pragma unroll
    for (int i = 0; i < 4; i++) o[i] = (T)(acc[i] / 3.0f);
    *reinterpret_cast<typename Op<T>::V4*>(out + tile_off(r, n, d >> 5)) = o;
  }
}

// fine row at position p: its own stream (the skip) plus the coarse output of slot floor(p/3)
template <typename T>
__global__ __launch_bounds__(256) void k_dec_upsample(float* __restrict__ h, const int* __restrict__ pos, int RPS,
                                                       const float* __restrict__ ring_coarse, int RSc, int d, T* __restrict__ xg,
                                                       const float* __restrict__ gain, float* __restrict__ ssq, const int* run_flag) {
  const int r = blockIdx.x, p = pos[r];
  if (*run_flag == 0) return;
  const float* c = ring_coarse + ((long)(r / RPS) * RSc + ((max(p, 0) / 3) & (RSc - 1))) * d;
  for (int n = threadIdx.x * 4; n < d; n += 1024) {
    f32x4 v = *reinterpret_cast<const f32x4*>(h + (long)r * d + n);
    if (p >= 0) v += *reinterpret_cast<const f32x4*>(c + n);
    put_row4(v, r, n, d, h, xg, gain, ssq);
  }
}

// ------------------------------------------------------------------------------------------
// Launch rules
// ------------------------------------------------------------------------------------------
template <typename T, int MT, int NC, int NW, int U, bool LOOP, int EPI, int NORM>
void dec_gemm_launch(const DecGemm& a, int groups, hipStream_t st) {
  const int tiles = (a.M + 15) / 16, NT = (a.N + 15) / 16;
  const size_t lds = (size_t)NW * MT * NC * 1024 + NW * MT * 64;
  if (lds > 65536) (void)hipFuncSetAttribute((const void*)k_dec_gemm<T, MT, NC, NW, U, LOOP, EPI, NORM>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  hipLaunchKernelGGL((k_dec_gemm<T, MT, NC, NW, U, LOOP, EPI, NORM>), dim3((NT + NC - 1) / NC, (tiles + MT - 1) / MT, groups), dim3(NW * 64), lds, st, a);
}

// Which tile a launch gets.  gridDim.x = column tiles comes first in the block order, so the row tiles of a column tile run on
// one die (the count of column tiles is a multiple of 8 for all weights but the output head's) and share its L2.
// Measured in a chain of dependent launches over cold weights (us; M rows, d = K of the first four):
//   M = 9, d = 1024: projection 3.7, up 4.5, down 6.8      M = 27, d = 768: 3.5, 4.4, 5.9
//   M = 72, d = 1024: 4.1, 6.7, 7.6                        M = 72, d = 1536: 5.1, 11.1, 11.7
template <typename T, int EPI, int NORM>
void dec_gemm(const DecGemm& a, int groups, hipStream_t st) {
  const int tiles = (a.M + 15) / 16, NT = (a.N + 15) / 16, KT = a.KT;
  const long wgs = (long)NT * tiles * groups;
  const bool pairs = NT % 2 == 0;
  if constexpr (std::is_same<T, float>::value) {
    // fp32: small models; operands take twice the registers
    if (tiles >= 8 && pairs) return dec_gemm_launch<T, 2, 2, 8, 2, true, EPI, NORM>(a, groups, st);
    return KT <= 32 ? dec_gemm_launch<T, 1, 1, 4, 8, false, EPI, NORM>(a, groups, st) : dec_gemm_launch<T, 1, 1, 8, 4, true, EPI, NORM>(a, groups, st);
  } else {
    // tall problems: operands shared by more of a workgroup's results, K in double-buffered chunks
    if (tiles >= 8 && pairs) return dec_gemm_launch<T, 4, 2, 8, 4, true, EPI, NORM>(a, groups, st);
    // K too long for one trip
    if (KT > 128) return wgs > 400 && pairs ? dec_gemm_launch<T, 1, 2, 8, 8, true, EPI, NORM>(a, groups, st) : dec_gemm_launch<T, 1, 1, 8, 8, true, EPI, NORM>(a, groups, st);
    // long K: 8 or 16 waves hold the whole K of their columns in flight
    if (KT > 64) return wgs > 200 && tiles >= 2 ? dec_gemm_launch<T, 2, 1, 16, 8, false, EPI, NORM>(a, groups, st) : dec_gemm_launch<T, 1, 1, 8, 16, false, EPI, NORM>(a, groups, st);
    // few workgroups: one tile each
    if (wgs <= 400 || !pairs) return dec_gemm_launch<T, 1, 1, 4, 16, false, EPI, NORM>(a, groups, st);
    // many: two column tiles share the activations
    return KT <= 32 ? dec_gemm_launch<T, 1, 2, 4, 8, false, EPI, NORM>(a, groups, st) : dec_gemm_launch<T, 1, 2, 8, 8, false, EPI, NORM>(a, groups, st);
  }
}

// GEMM whose workgroups norm their rows themselves (DN_ROWS); false: not for this size.  A lane holds rows and gains as fp32 beside the weights, up to
// eight fragments of each (four waves up to K = 1024, eight up to 2048; fp32 up to 1024).  For one row tile and few workgroups: each of them
// reads twice the bytes of rows in operand order, and gains.  Steps with the norm inside / in a launch of its own, us: d = 512 one sequence
// 575 / 579, d = 768 three 1182 / 1188, d = 1024 one 1436 / 1435, a mesh of d = 256 fp32 10 480 / 10 580; for all sizes (with the factor on the result, a barrier less)
// d = 2048 2270 / 2210, eight sequences of d = 1024 3196 / 3184.
template <typename T, int EPI>
bool dec_gemm_rows(const DecGemm& a, int groups, hipStream_t st) {
  if (a.M > 16 || (long)((a.N + 15) / 16) * groups > 400 || a.KT > (std::is_same<T, float>::value ? 32 : 64)) return false;
  if (a.KT <= 32) dec_gemm_launch<T, 1, 1, 4, 8, false, EPI, DN_ROWS>(a, groups, st);
  else if constexpr (!std::is_same<T, float>::value) dec_gemm_launch<T, 1, 1, 8, 8, false, EPI, DN_ROWS>(a, groups, st);
  return true;
}

// Splits of an attention launch over `pairs` (head, sequence, set) triples: at most one workgroup of eight waves per compute
// unit (256), a number of workgroups that divides them unevenly costs more than idle ones: with 96 pairs (d = 1536, 4
// sequences) the step takes 4186 us with 2 splits, 4603 with 3, 4410 with 5; with 128 pairs 3231 with 2, 3475 with 3, 3423 with 4.
inline int attn_splits(long pairs, int capb, int NW) {
  const long ns = pairs < 256 ? 256 / pairs : 1;
  const int most = (capb + NW - 1) / NW;
  return (int)(ns > most ? most : ns);
}
inline size_t attn_ws_floats(int H, int S, int sets, int hd) {
  const long pairs = (long)H * S * sets;      // pairs * splits < 2048 / 8 + pairs, parts of up to 32 rows
  return (size_t)(256 + pairs) * (32 * hd + 64);
}

// Whether a launch loads its keys and values as read once (non-temporal), so that they do not push the weights that the readers have fetched, and the rows between
// the launches, out of L2: where its own caches hold 5 MB or more (L2 has 4 MB a die), as they are allocated: how much of them is in use only the device
// knows.  Two sets over one cache count once.  Steps without / with the hint, us.  By the memory's keys and values of a block:
//   134 MB (eight sequences of d = 1024) 3191 / 3086     101 MB (four, 1536) 4083 / 3964        75 MB (twelve, 768) 1232 / 1211
//   34 MB (one, 2048, heads of 128) 2225 / 2216          17 MB (four, 512) 450 / 431            17 MB (four, 256) 905 / 852
//   13 MB (twelve, 512) 916 / 909                        8 MB (five, 512, 20 faces sampled) 56.3 / 53.2 ms, (one, 1024, heads of 128) 1197 / 1200
//   6 MB (two, 768) 1052 / 1050, (one, 1536) 1303 / 1305   4 MB (two, 512) 879 / 881
//   1 MB (two, 512) 780 / 783, (two, 256, token by token) 29.37 / 30.47 ms: there L2 keeps them from pass to pass
// By the self-attention's at the coordinate level, memory of 0.5 to 4 MB a block: 147 MB (eight, 1024) 1372 / 1355     18 MB (two, 512) 835 / 787
//   15 MB (four, 512) 747 / 743     74 MB, the most 0.8 in use (two, 512, 20 faces with room for 2000) 18.55 / 17.17 ms
//   37 MB, the most 0.2 in use (two, 256, 8 faces token by token with room for 2000) 15.70 / 15.81 ms
//   and with 25 to 67 MB of memory a block, hinted or not:  4 MB (eight, 512) 971 / 974     1 MB (three, 256) 313 / 316
// The same hint on the weights of k_dec_gemm, whose row tiles share them: 3964 -> 4086 for four sequences of d = 1536.
template <class SET>
bool attn_once(const SET* set, int nset, int S, int H, int hd) {
  double bytes = 0;
  for (int z = 0; z < nset; z++)
    if (z == 0 || set[z].Kc != set[z - 1].Kc) bytes += 2.0 * 2.0 * S * set[z].capb * 32 * H * hd;
  return bytes >= 5e6;
}

template <typename T, int QT, int HD, int NW, bool ONCE>
void dec_attn_go(const AttnArgs& a, int nset, hipStream_t st) {
  const size_t lds = ((size_t)NW * QT * 16 * (HD + 4) + 2 * NW * QT * 16) * 4;
  if (lds > 65536) (void)hipFuncSetAttribute((const void*)k_dec_attn<T, QT, HD, NW, ONCE>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  hipLaunchKernelGGL((k_dec_attn<T, QT, HD, NW, ONCE>), dim3(a.H, a.ns_max, a.S * nset + a.ahead), dim3(NW * 64), lds, st, a);
}

template <typename T, int QT, int HD, int NW, bool ONCE = false>
void dec_attn_sized(AttnArgs& a, int nset, hipStream_t st) {
  a.ns_max = 1;
  for (int z = 0; z < nset; z++) {
    a.set[z].ns = attn_splits((long)a.H * a.S * nset, a.set[z].capb, NW);
    if (a.set[z].ns > a.ns_max) a.ns_max = a.set[z].ns;
  }
  a.nset = nset;
  // Readers come in whole planes of H * ns_max workgroups, 48 of them or more (32 to 128: no difference): 48 to 256.  Where one workgroup
  // that attends fills a compute unit (two tiles of 128-wide heads: 137 KB of LDS) and these fill the chip, the readers run behind them.
  a.ahead = a.next[0].W ? (48 + a.H * a.ns_max - 1) / (a.H * a.ns_max) : 0;
  dec_attn_go<T, QT, HD, NW, ONCE>(a, nset, st);
}
// Waves of a workgroup: 8, in fp32, whose operands take twice the registers, 4.  Over at most 16 key blocks fp32 takes two, a wave for each block on
// two to four times as many compute units: one of them pulls about 55 KB a microsecond and a block of a 64-wide head is 16 KB (a mesh of ten
// faces, d = 256, memory 256: 10.91 -> 10.53 ms; with eight waves 11.05).  Past 16 blocks that is more than the 8 parts which the merge reads in one
// trip, and costs more than it gives (one sequence, 600 faces, two heads of 128: 805 us a step, 935 with two waves over any number of blocks).
// Half precision with four waves instead of eight: d = 768, three sequences 1170 -> 1198 us a step.
template <typename T, int QT, int HD>
void dec_attn_waves(AttnArgs& a, int nset, hipStream_t st) {
  int blocks = 0;
  for (int z = 0; z < nset; z++) blocks = a.set[z].capb > blocks ? a.set[z].capb : blocks;
  if constexpr (std::is_same<T, float>::value) {
    if (blocks <= 16 && (long)a.H * a.S * nset * ((blocks + 1) / 2) <= 256) dec_attn_sized<T, QT, HD, 2>(a, nset, st);
    else dec_attn_sized<T, QT, HD, 4>(a, nset, st);
  } else {
    if (attn_once(a.set, nset, a.S, a.H, HD)) dec_attn_sized<T, QT, HD, 8, true>(a, nset, st);
    else dec_attn_sized<T, QT, HD, 8>(a, nset, st);
  }
}
// Attention of `nset` row sets (at most 32 rows each) in one launch.
template <typename T>
bool dec_attention(AttnArgs& a, int nset, int hd, hipStream_t st) {
  int QT = 1;
  for (int z = 0; z < nset; z++) {
    if (a.set[z].rows > 32) return false;
    if (a.set[z].rows > 16) QT = 2;
  }
  if (hd == 64) { if (QT == 1) dec_attn_waves<T, 1, 64>(a, nset, st); else dec_attn_waves<T, 2, 64>(a, nset, st); }
  else if (hd == 96) { if (QT == 1) dec_attn_waves<T, 1, 96>(a, nset, st); else dec_attn_waves<T, 2, 96>(a, nset, st); }
  else { if (QT == 1) dec_attn_waves<T, 1, 128>(a, nset, st); else dec_attn_waves<T, 2, 128>(a, nset, st); }
  return true;
}
