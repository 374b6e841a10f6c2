// Persistent verify kernel for the half-precision path, one sequence, blocks of up to 32 tokens: the whole backbone
// forward of one verify pass is ONE launch.  Rows are handled in groups of 16 (one MFMA row tile): blocks of up to
// 16 tokens have one group per level, longer ones two at the coordinate level (template parameter QT).
//
// Why: at batch 1 a transformer block is ~10 dependent operations of 0.3-1 us of HBM time each; as
// separate launches every one costs ~4 us.  Here 256 resident workgroups walk a static schedule of
// stages (GEMM tiles, attention splits, merges, level transitions) and hand activations to each other
// through "tagged" exchange buffers: every 8-byte element carries 4 bytes of payload and a 4-byte tag
// (launch epoch, layer).  A consumer simply re-reads an element until its tag is the one it expects, so
// correctness never depends on the order in which stores become visible across XCDs, and there is no
// grid barrier.  Elements are written with agent-scope 8-byte atomic stores and read with agent-scope loads
// (8-byte atomics for single elements, 16-byte loads of two elements for bulk reads: each element still
// arrives whole), which bypass the per-XCD L2, not coherent across XCDs inside a launch.
// A workgroup that is not needed in a stage runs ahead and issues the weight loads of its next tile
// before it starts waiting, which is what keeps HBM busy across the dependency chain.
//
// Every wait is bounded (wall clock); on a time-out the kernel raises an abort word that every waiter
// polls, so all workgroups leave and the host reports an error instead of hanging.
//
// Arithmetic is kept batch-invariant exactly like the per-launch kernels: fixed 32-key blocks, fixed
// deal of the blocks to the splits, fixed merge order, rows never mixed in a GEMM.
#pragma once
#include "fm_device.h"
#include "fm_kernels_mfma.h"
#include "fm_kernels_step.h"
#include "fm_transition.h"

typedef unsigned long long u64;

#define PK_NWG 256
#define PK_MAXSPLIT 16                    // parts that a merge unit takes in one round of loads
#define PK_PART (16 * 64 + 32)            // per (head, split): 16x64 unnormalised O, 16 pairs of running maximum and sum
#define PK_TIMEOUT_TICKS 20000000ull      // default bound of every wait: 200 ms of the 100 MHz wall clock

// A pointer read from a table in memory is generic to the compiler, and loads through it become FLAT instructions,
// which count against the LDS counter as well: every wait for an LDS read would then also wait for the weight
// or cache loads in flight.  The table therefore holds pointers that are typed as global.
#define PK_GLOBAL __attribute__((address_space(1)))
typedef const PK_GLOBAL f16_t* pk_cw_t;     // weights, condition-memory caches
typedef PK_GLOBAL f16_t* pk_w_t;            // self-attention caches (appended to by this kernel)
typedef const PK_GLOBAL float* pk_cf_t;     // gains

struct PkLayer {
  pk_cf_t g1, g2, g3;
  pk_cw_t wqkv, wo, cq, co, w1, w2;   // tiled; wqkv with rotary pairs inside one tile
  pk_w_t Kc, Vc;
  pk_cw_t Km, Vm;
  int level;      // 0 coordinate, 1 vertex, 2 face
  int tap;        // store the layer input to the level's tap ring (input of the last layer of a stack)
  int last;       // last layer of its stack: output goes to hT[stack] and to the stack's ring
  int stack;      // 0 cpre, 1 vpre, 2 face, 3 vpost, 4 cpost
};

// Width of the model: FWT fragments of 32 per wave in a GEMM over d, i.e. d = 128 FWT, known to the compiler for some widths (pk_kernel;
// the hidden width is then 4 d), read from the arguments for the others (FWT = 0).
struct PkArgs;
template <int FWT> __device__ __forceinline__ int pk_d(const PkArgs& a);

struct PkArgs {
  const PkLayer* layers;
  int n_layers;
  int first[5], count[5];
  Dims D;
  int ff;
  float eps;
  int R[3];                 // row slots per level (<= RS)
  int RS;                   // rows the exchange buffers hold per region: 16, or 32 when the coordinate level has two row groups
  int capb[3], capbM;       // cache capacity in 32-key blocks per level / of the condition memory
  int nsplit[3], nsplitM;   // launch-time split counts (fixed partition of the key axis)
  int win[3];               // sliding window per level (0 = none); the self-attention caches are then rings of capb blocks
  const int* pos[3];
  const int* limx[3];
  const float2* cs[3];
  const int* vtok;
  float *ring_hc, *ring_hv, *ring_yf, *ring_yv;
  float* tap[3];
  const f16_t *emb, *short_cv, *short_vf, *lm;
  const float* gf;
  float* logits;
  // exchange buffers (u64 = payload | tag << 32)
  u64 *hA, *hB, *hC;        // [layers + 1][RS][d]: one region per layer, written once per launch
  u64* hT[4];               // outputs of cpre, vpre, face, vpost  [RS][d]
  u64 *xA, *xB, *xC;        // [layers (+ 1)][RS][d/2]: half(row of hA, hB, hC times the gain of the norm that reads it), pairs
  u64 *sA, *sB, *sC;        // [layers (+ 1)][RS][d/16]: sums of squares of 16 columns of those rows
  u64 *q, *q2;              // [RS][d/2] rotated queries of the self- / cross-attention (half pairs)
  u64 *att, *att2;          // [layers][RS][d/2] attention outputs
  u64* pool;                // [2][16][d/2] pooled groups before the two shortening projections (coarse rows: at most 9)
  u64* mid;                 // [layers][RS][ff/2]
  u64 *newK, *newV;         // [H][RS][32]
  u64 *partS, *partX;       // [H][PK_MAXSPLIT][RS/16][PK_PART]
  u64* w2part;              // [d/16][RS/16][3][256]: partial tiles of the K-quarters 1..3 of the FFN down projection
  const unsigned* epoch_word;  // passes so far, counted by k_verify_setup
  u64 timeout_ticks;        // bound of every wait (100 MHz wall clock)
  unsigned test_skew;       // test hook: added to the tag the embedding publishes, so that nothing downstream ever arrives
  unsigned* abort_word;     // [0] abort flag, [1] earliest stage that gave up, [2] claim, [3..8] expected tag, tag seen,
                            // stage, workgroup, thread, element of the first missing value
  const int* run_flag;
  int prof_stage;           // stage whose inner phases are timed into prof[600..]
  u64* prof;                // optional [1 + stages]: earliest start, latest completion per stage (wall clock ticks)
};

template <int FWT> __device__ __forceinline__ int pk_d(const PkArgs& a) { return FWT ? FWT * 128 : a.D.d; }

// Exchanges between the waves of a workgroup.  Two sets, used by the GEMM and attention units in turn: a unit writes its set, passes its one
// barrier and reads; who writes the same set two units later has passed the barrier between, so all have read.
template <int QT>
struct PkShared {
  float red[2][4][4][64];
  float ssq[2][4][16];
  __align__(16) float lo[2][4][16 * QT][68];
  float lm[2][4][16 * QT], ll[2][4][16 * QT];
  int bad;                  // raised by a wave whose wait gave up
};

// Barrier at which all waves learn whether one of them has given up.  (__syncthreads_or is three barriers and two trips to LDS, in
// every unit: steps of 755 us at d = 512 and 1817 us at d = 1024 become 728 and 1755.)
template <class SH>
__device__ __forceinline__ bool pk_sync(SH& sh, bool good) {
  if (!good) sh.bad = 1;
  __syncthreads();
  return sh.bad == 0;
}

__device__ __forceinline__ u64 pk_ld(const u64* p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void pk_st(u64* p, unsigned payload, unsigned tag) {
  __hip_atomic_store(p, ((u64)tag << 32) | payload, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void pk_stf(u64* p, float v, unsigned tag) { pk_st(p, __float_as_uint(v), tag); }
__device__ __forceinline__ unsigned pk_pack(float lo, float hi) {
  const f16_t a = (f16_t)lo, b = (f16_t)hi;
  return (unsigned)__builtin_bit_cast(unsigned short, a) | ((unsigned)__builtin_bit_cast(unsigned short, b) << 16);
}
__device__ __forceinline__ bool pk_expired(const PkArgs& a, u64 t0, int stage) {
  // every waiter that gives up records its stage; the smallest one is where the chain broke
  if (__hip_atomic_load(a.abort_word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
    atomicMin(a.abort_word + 1, (unsigned)stage);
    return true;
  }
  if (wall_clock64() - t0 > a.timeout_ticks) {
    __hip_atomic_store(a.abort_word, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    atomicMin(a.abort_word + 1, (unsigned)stage);
    return true;
  }
  return false;
}

// Wave-wide fetch of N tagged elements per lane (addresses from `addr(i)`, i < n <= N); inactive lanes get 0.
// All loads are issued before any is checked; the whole set is re-read until every tag matches.  (Watching one element first costs a
// second trip once it is there: 40 us of a step at d = 1024.  The abort word is another trip, so it is looked at every 64 rounds only.)
template <int N, class F>
__device__ __forceinline__ bool pk_fetch(unsigned (&out)[N], int n, bool active, unsigned tag, F addr, const PkArgs& a, int stage) {
  const u64 t0 = wall_clock64();
  int it = 0;
  while (true) {
    // all loads are issued back to back (the compiler keeps agent-scope loads in program order and would
    // otherwise wait for each one before the next), only then are the tags looked at
    u64 v[N];
#pragma unroll
    for (int i = 0; i < N; i++) {
      v[i] = 0;
      if (active && i < n) v[i] = pk_ld(addr(i));
    }
    bool ok = true;
#pragma unroll
    for (int i = 0; i < N; i++) {
      out[i] = (unsigned)v[i];
      if (active && i < n) ok = ok && ((unsigned)(v[i] >> 32) == tag);
    }
    if (__all(ok)) return true;
    if ((++it & 63) == 0 && pk_expired(a, t0, stage)) {
      // diagnostics of the first element found missing: expected tag, tag seen, stage, workgroup, thread
      if (!ok && atomicCAS(a.abort_word + 2, 0u, 1u) == 0u) {
        unsigned seen = 0, idx = 0;
        for (int i = 0; i < N; i++)
          if (active && i < n) { const u64 v = pk_ld(addr(i)); if ((unsigned)(v >> 32) != tag) { seen = (unsigned)(v >> 32); idx = i; break; } }
        a.abort_word[3] = tag; a.abort_word[4] = seen; a.abort_word[5] = (unsigned)stage;
        a.abort_word[6] = blockIdx.x; a.abort_word[7] = threadIdx.x; a.abort_word[8] = idx;
      }
      return false;
    }
    __builtin_amdgcn_s_sleep(1);
  }
}

#define PK_TAG(l) (epoch * 64u + (unsigned)(l) + 1u)      // epoch: local of the kernel

// A level transition must not publish anything before the stack below it has finished with the shared
// exchange buffers, even when its own rows are inactive or only need data of earlier passes: it first
// waits for the stack output from EVERY tile, the first row of each of the tile's four waves (wave w stores rows w, w + 4, ...
// behind its last read, of the partial tiles of the FFN down projection, and no barrier follows that one).  All in one trip.
// No barrier stands between this wait and what the unit publishes.  Hence COLS (fm_transition.h): a thread waits for the columns that it then
// publishes; who needs the row of the unit needs all its columns, and so all tiles have been waited for.
// The rows of the stack that the unit needs (`row(k)`, k < OWN) come in the same trip, the thread's columns of row k in
// got[k].  (Each element in a trip of its own: upsampling 4.4 us
// instead of 2.2 at d = 512, 8.0 instead of 3.4 at 1024; pooling 4.9 instead of 2.9 there.)
template <int FWT, class COLS, int OWN, class ROW>
__device__ __forceinline__ bool pk_wait_stack(const PkArgs& a, const u64* hT, unsigned tag, int stage, int rows, ROW row, float (&got)[OWN][FM_TR_COLS]) {
  const int d = pk_d<FWT>(a);
  const int n = COLS::count(d, threadIdx.x);
  const agent_buf_t hb = agent_buf(hT, rows * d * 8);
  u32x2 own[OWN][FM_TR_COLS];
  bool ok = true;
  for (int r0 = 0; r0 < rows && ok; r0 += 16) {               // a second row group is written by units of its own
    const u64 t0 = wall_clock64();
    int it = 0;
    while (true) {
      agent_again();
      u32x2 seen[4][FM_TR_COLS];
      unsigned diff = 0;
#pragma unroll
      for (int c = 0; c < FM_TR_COLS; c++) {
        const int col = COLS::col(threadIdx.x, min(c, max(n - 1, 0)));      // columns that the thread does not have: its last one again
#pragma unroll
        for (int k = 0; k < 4; k++) seen[k][c] = ld_agent2(hb, ((r0 + min(k, rows - r0 - 1)) * d + col) * 8);
#pragma unroll
        for (int k = 0; k < OWN; k++) own[k][c] = ld_agent2(hb, (row(k) * d + col) * 8);
      }
#pragma unroll
      for (int c = 0; c < FM_TR_COLS; c++) {
#pragma unroll
        for (int k = 0; k < 4; k++) diff |= seen[k][c][1] ^ tag;
#pragma unroll
        for (int k = 0; k < OWN; k++) diff |= own[k][c][1] ^ tag;
      }
      if (__all(diff == 0 || n <= 0)) break;
      if ((++it & 63) == 0 && pk_expired(a, t0, stage)) { ok = false; break; }
      __builtin_amdgcn_s_sleep(1);
    }
  }
#pragma unroll
  for (int k = 0; k < OWN; k++)
#pragma unroll
    for (int c = 0; c < FM_TR_COLS; c++) got[k][c] = __uint_as_float(own[k][c][0]);
  return ok;
}

// Times of a stage (debug), the latest of all waves: each of them finishes a quarter of a unit, and no barrier follows.
#define PK_STAMP(i) do { if ((threadIdx.x & 63) == 0) atomicMax(a.prof + (i), (u64)wall_clock64()); } while (0)
// phase timing inside the units of one chosen stage: latest time each phase was reached
#define PK_MARK(k) do { if (a.prof && stage == a.prof_stage) PK_STAMP(600 + (k)); } while (0)

// ------------------------------------------------------------------------------------------
// GEMM tile: C[16 rows x 16 cols] = A[16 x K] * W_tile^T, four waves split K (K <= 1024).  Behind the one barrier of the unit every wave
// owns a quarter of the result: wave w of lane (g, col) has row g*4 + w, column col in `result`.
// A is a half-pair exchange buffer [16][K/2].  NORM: its rows are half(x * gain), written so by the producers of the residual stream
// together with the sums of squares of every 16 columns, sq[row][K/16]; the row factor 1/rms goes onto the result.
// (One wave doing the whole epilogue, and gain and sums computed here: steps of 707 us at d = 512 and 1692 us at d = 1024, against 644 and
// 1526 with the merge below.)
// Every wave takes the MFMA A-fragments of its K-quarter straight from the exchange buffer: lane (r, g) of
// fragment f needs the 8 consecutive values k0 = f*32 + g*8 .. +8 of row r, which are 32 contiguous bytes of
// tagged half pairs, i.e. two 16-byte agent-scope loads.  No LDS staging, no barrier before the multiplication;
// the tags are checked per lane and the whole set is re-read until complete.
// ------------------------------------------------------------------------------------------
template <int FWT, bool NORM, class SH>
__device__ __forceinline__ bool pk_gemm_tile(const PkArgs& a, SH& sh, int& par, pk_cw_t Wt, int KT, const u64* A,
                                             unsigned tagA, const u64* sq, int R, float& result, int stage, int lda = 0) {
  constexpr int NL = 2;       // 16-byte loads per fragment and lane
  constexpr int EF = 16;      // tagged elements (half pairs) per fragment row
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int r = lane & 15, g = lane >> 4;
  const bool on = r < R;
  constexpr int NF = FWT ? FWT : 8;
  const int FW = FWT ? FWT : KT >> 2;      // fragments per wave (host guarantees KT % 4 == 0, KT <= 32)
  const int K = FW * 128;
  if (lda == 0) lda = K >> 1;
  par ^= 1;
  f32x4 acc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
  // weights go out before the wait for the activations: they depend on nothing
  f16x8 wf[NF];
#pragma unroll
  for (int f = 0; f < NF; f++)
    if (f < FW) wf[f] = *(const PK_GLOBAL f16x8*)(Wt + ((long)(wave * FW + f) * 64 + lane) * 8);
  // this wave's part of the rows: element (wave*FW + f)*EF + g*(EF/4) of row r is where fragment f starts; rows past the last lie outside the
  // buffer and read 0 (a branch around every load instead: step of d = 1024 1810 -> 1907 us, d = 512 761 -> 805)
  const agent_buf_t Ab = agent_buf(A, ((R - 1) * lda + KT * EF) * 8);
  const int mine = on ? (r * lda + (wave * FW) * EF + g * (EF / 4)) * 8 : 1 << 30;
  // sums of squares of the columns of this K-quarter: pair p of 16-column sums belongs to fragment p, lane (r, g) takes p = g and g + 4
  const agent_buf_t Sb = agent_buf(NORM ? sq : A, NORM ? R * FW * 8 * 8 : 0);
  const bool son[2] = {on && g < FW, on && g + 4 < FW};
  int so[2];
#pragma unroll
  for (int j = 0; j < 2; j++) so[j] = son[j] ? ((r * 4 + wave) * FW + g + 4 * j) * 16 : 1 << 30;
  const u64 t0 = wall_clock64();
  int it = 0;
  bool good = true;
  // The full fragment read is its own validity check, so a unit whose input is already there pays one round trip.
  // When a read comes back incomplete the wave falls back to watching one element per lane (lane l: fragment l/8, its
  // first or second half - a producer tile owns half a fragment row - in one of the last four rows) and reads the
  // fragments again once those show the tag: waiting costs the memory system 64 small loads per round, not 32 KiB (reading all
  // again instead, steps in us: d = 1024 1893 -> 1905, d = 512 800 -> 810; for up to four rows only: 1904, 805).
  const int fs_ = min(lane >> 3, FW - 1), hs_ = (lane >> 2) & 1, rs_ = max(R - 1 - (lane & 3), 0);
  const u64* watched = A + (long)(wave * FW) * EF + (long)rs_ * lda + fs_ * EF + hs_ * (EF / 2);
  PK_MARK(1);
  u32x4 v[NF * NL], sv[2];
  while (good) {
    agent_again();
#pragma unroll
    for (int f = 0; f < NF; f++)
      if (f < FW)
#pragma unroll
        for (int j = 0; j < NL; j++) v[f * NL + j] = ld_agent4(Ab, mine + (f * EF + 2 * j) * 8);
    if (NORM) {
      sv[0] = ld_agent4(Sb, so[0]);
      if (NF > 4) sv[1] = ld_agent4(Sb, so[1]);
    }
    unsigned diff = 0;
#pragma unroll
    for (int f = 0; f < NF; f++)
      if (f < FW)
#pragma unroll
        for (int j = 0; j < NL; j++) diff |= (v[f * NL + j][1] ^ tagA) | (v[f * NL + j][3] ^ tagA);
    if (NORM) {
      if (son[0]) diff |= (sv[0][1] ^ tagA) | (sv[0][3] ^ tagA);
      if (NF > 4 && son[1]) diff |= (sv[1][1] ^ tagA) | (sv[1][3] ^ tagA);
    }
    if (__all(diff == 0 || !on)) break;
    if ((++it & 63) == 0 && pk_expired(a, t0, stage)) { good = false; break; }
    while (!__all((unsigned)(pk_ld(watched) >> 32) == tagA)) {
      if ((++it & 63) == 0 && pk_expired(a, t0, stage)) { good = false; break; }
      __builtin_amdgcn_s_sleep(1);
    }
  }
  PK_MARK(2);
#pragma unroll
  for (int f = 0; f < NF; f++) {
    if (f < FW) {
      const u32x4 pk = {v[2 * f][0], v[2 * f][2], v[2 * f + 1][0], v[2 * f + 1][2]};
      acc[f & 1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, pk), wf[f], acc[f & 1], 0, 0, 0);
    }
  }
  if (NORM) {       // what lies outside the buffer has read 0
    float ss = __uint_as_float(sv[0][0]) + __uint_as_float(sv[0][2]);
    if (NF > 4) ss += __uint_as_float(sv[1][0]) + __uint_as_float(sv[1][2]);
    ss = rows_sum(ss);
    if (g == 0) sh.ssq[par][wave][r] = ss;
  }
  acc[0] += acc[1];
#pragma unroll
  for (int i = 0; i < 4; i++) sh.red[par][wave][i][lane] = acc[0][i];
  if (!pk_sync(sh, good)) return false;
  PK_MARK(3);
  result = sh.red[par][0][wave][lane] + sh.red[par][1][wave][lane] + sh.red[par][2][wave][lane] + sh.red[par][3][wave][lane];
  if (NORM) {
    const int row = g * 4 + wave;
    const float tot = sh.ssq[par][0][row] + sh.ssq[par][1][row] + sh.ssq[par][2][row] + sh.ssq[par][3][row];
    result *= 1.0f / sqrtf(tot / (float)K + a.eps);
  }
  return true;
}

// Epilogues: a thread has row g*4 + wave (wave, lane as above) and column n = nt*16 + lane%16 of the tile.

// One value of a row of the residual stream: the value, half(value * gain of the norm that reads it) and, per 16 columns, the sum of squares.
// x null: no norm reads this row.
__device__ __forceinline__ void pk_put_row(float v, bool on, int row, int n, int d, u64* h, u64* x, u64* sq, float gain, unsigned tag) {
  const float xg = v * gain, w = lane_xor1(xg), ss = row16_sum(v * v);
  if (!on) return;
  if (x) {
    if ((n & 1) == 0) pk_st(x + (long)row * (d >> 1) + (n >> 1), pk_pack(xg, w), tag);
    if ((n & 15) == 0) pk_stf(sq + (long)row * (d >> 4) + (n >> 4), ss, tag);
  }
  pk_stf(h + (long)row * d + n, v, tag);
}

// The residual operand of a tile (complete long before the tile's GEMM input is) is requested at the start of the unit and looked at behind
// the multiplication; only then, if it was not there yet, it is waited for.
struct PkOld { u32x2 v; int p; float gain; };
template <int FWT>
__device__ __forceinline__ void pk_res_request(const PkArgs& a, int n, const u64* hold, int R, const int* pos, pk_cf_t gain, PkOld& o) {
  const int d = pk_d<FWT>(a), row = min(((threadIdx.x & 63) >> 4) * 4 + (int)(threadIdx.x >> 6), R - 1);
  o.v = ld_agent2(agent_buf(hold, R * d * 8), (row * d + n) * 8);
  o.p = pos[row];
  o.gain = gain ? gain[n] : 0.f;
}
template <int FWT>
__device__ __forceinline__ bool pk_res_take(const PkArgs& a, int n, const u64* hold, unsigned tag, int R, const PkOld& o, float& old, int stage) {
  const int d = pk_d<FWT>(a), row = min(((threadIdx.x & 63) >> 4) * 4 + (int)(threadIdx.x >> 6), R - 1);
  unsigned raw[1] = {o.v[0]};
  bool ok = true;
  if (!__all(o.v[1] == tag)) ok = pk_fetch<1>(raw, 1, true, tag, [&](int) { return hold + (long)row * d + n; }, a, stage);
  old = __uint_as_float(raw[0]);
  return ok;
}

// dst[row][n/2] = (c[n], c[n+1]) as halves
__device__ __forceinline__ void pk_put_half(float v, bool on, int row, int n, u64* dst, int ld2, unsigned tag) {
  const float w = lane_xor1(v);
  if (on && (n & 1) == 0) pk_st(dst + (long)row * ld2 + (n >> 1), pk_pack(v, w), tag);
}

// QKV epilogue.  Tiles of the q and k parts hold 8 rotary pairs: columns 0..7 = dims qd*8.., columns
// 8..15 = the same dims + 32.  q -> exchange buffer; k, v -> cache (for later passes) and exchange buffers.
struct PkQkvPre {     // what the QKV epilogue needs besides the tile: requested before the tile's input arrives
  float2 t;           // rotary (cos, sin) of the thread's pair in its row
  int p;              // position of that row
};
__device__ __forceinline__ void pk_qkv_prefetch(int nt, int d, int R, const int* pos, const float2* cs, PkQkvPre& pre) {
  const int lane = threadIdx.x & 63, col = lane & 15, rr = min((lane >> 4) * 4 + (int)(threadIdx.x >> 6), R - 1);
  const int part = (nt * 16) / d, cp = (nt * 16) % d;
  const int qd = (cp & 63) >> 4;
  pre.p = pos[rr];
  pre.t = part < 2 ? cs[(long)rr * 32 + qd * 8 + (col & 7)] : float2{1.f, 0.f};
}
template <int QT, int FWT>
__device__ __forceinline__ void pk_epi_qkv(const PkArgs& a, const PkLayer& L, float v, int nt, unsigned tag, int R,
                                           const PkQkvPre& pre, int capb, int row0) {
  const int lane = threadIdx.x & 63, col = lane & 15, r = (lane >> 4) * 4 + (int)(threadIdx.x >> 6);
  const int d = pk_d<FWT>(a);
  const int part = (nt * 16) / d, cp = (nt * 16) % d;
  const int hh = cp >> 6, qd = (cp & 63) >> 4;
  int dim = qd * 16 + col;
  if (part < 2) {
    const float o = lane_xor8(v);
    v = col < 8 ? v * pre.t.x - o * pre.t.y : v * pre.t.x + o * pre.t.y;
    dim = (col < 8 ? 0 : 32) + qd * 8 + (col & 7);
  }
  const float w = lane_xor1(v);       // neighbour dim (dim ^ 1 sits in lane ^ 1 in every layout above)
  if (r >= R) return;
  if (part == 0) {
    if ((lane & 1) == 0) pk_st(a.q + (long)(row0 + r) * (d >> 1) + ((hh * 64 + dim) >> 1), pk_pack(v, w), tag);
  } else {
    u64* nb = (part == 1 ? a.newK : a.newV) + ((long)hh * (QT * 16) + row0 + r) * 32;
    if ((lane & 1) == 0) pk_st(nb + (dim >> 1), pk_pack(v, w), tag);
    if (pre.p >= 0) {
      const int ps = pre.p % (capb * 32);      // the cache is a ring when a window is set
      const long base = (long)hh * capb * 2048;
      if (part == 1) L.Kc[base + kblk_off(ps, dim)] = (f16_t)v;
      else L.Vc[base + vblk_off(ps, dim)] = (f16_t)v;
    }
  }
}

__device__ __forceinline__ int pk_active(int nblk, int ns) { return max(1, min(ns, (nblk + 3) >> 2)); }      // splits that hold visible keys
__device__ __forceinline__ int pk_parts(int maxlim, int capb, int ns) {      // and so parts per head, uniform
  return __builtin_amdgcn_readfirstlane(pk_active(min((maxlim + 32) >> 5, capb), ns));
}

// ------------------------------------------------------------------------------------------
// Attention over one split of the keys of one head (flash-decoding), same arithmetic and deal as k_dec_attn: block b of 32 keys
// belongs to wave b % 4 of split (b / 4) % ns, which is balanced at every length and does not depend on it.  QT tiles of
// 16 query rows share every K/V block that is loaded.  The first K/V block of a wave is requested before the wait for
// the queries, the next one behind it.  Keys of this pass (positions >= P0) are taken from the
// exchange buffers, older keys from the cache.  lim[t]: last key the lane's row of tile t may see (-1: unused slot).
// Partial results: tile t of (head, split) at part + t * PK_PART.  Where one split holds all visible keys (contexts of up to 128) there is nothing
// to merge: its unit writes the attention output, and the merge stage, an exchange of 1.1 to 2 us, is left
// out (eight faces token by token at d = 512, with the trips above: 29.9 -> 26.3 ms).
// ------------------------------------------------------------------------------------------
template <int QT, int FWT, class SH>
__device__ __forceinline__ bool pk_attn_unit(const PkArgs& a, SH& sh, int& par, const u64* qbuf, const int (&lim)[QT], int maxlim, int R,
                                             pk_cw_t Kc, pk_cw_t Vc, int capb, int nsplit_cfg, int hh, int split,
                                             bool overlay, int P0, u64* part, u64* att, unsigned tag, int stage, int window) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int g = lane >> 4, ql = lane & 15;
  const int d = pk_d<FWT>(a);
  const float kScale = 0.125f * 1.4426950408889634f;
  // With a window the cache is a ring of capb blocks (a multiple of four): position p lives in slot p mod (32 capb);
  // seen from the newest visible position, slot j holds lapbase + j if that is <= maxlim, else the position one
  // lap earlier.  Without a window lapbase = 0 and nothing wraps.
  maxlim = __builtin_amdgcn_readfirstlane(maxlim);
  const int nblk = min((maxlim + 32) >> 5, capb);
  const int ringn = capb * 32;
  const int lapbase = max(maxlim, 0) / ringn * ringn;
  auto held = [&](int slot) { const int k = lapbase + slot; return k > maxlim ? k - ringn : k; };
  bool on[QT];
  int first[QT];
#pragma unroll
  for (int t = 0; t < QT; t++) {
    on[t] = t * 16 + ql < R;
    first[t] = window > 0 ? max(lim[t] - window + 1, 0) : 0;
  }
  const int nact = pk_active(nblk, nsplit_cfg);
  if (split >= nact) return true;      // nothing visible in this split: the merge knows the same count
  par ^= 1;
  const int b0 = split * 4 + wave, step = nsplit_cfg * 4;     // this wave's blocks: b0, b0 + step, ...

  // The block of this wave, if any, that holds rows written by this pass.  K fragment f = (hb, dh) holds key b*32 + hb*16 + lane%16, dims
  // dh*32 + g*8..+8 (4 elements); V fragment dt holds dim dt*16 + lane%16 and the 8 slots g*8 + j <-> key b*32 + (j/4)*16 + g*4 + j%4.
  int bov = -1;
  if (overlay) {
    // slot blocks of the rows of this pass: neighbours (also around a ring, whose blocks are a multiple of four), so in different waves;
    // rows past the end of a cache that is no ring do not exist
    const int end = window > 0 ? (P0 + R - 1) % ringn : min(P0 + R - 1, ringn - 1);
    const int cand[2] = {(P0 % ringn) >> 5, end >> 5};
#pragma unroll
    for (int k = 0; k < 2; k++) {
      const int b = cand[k];
      if (b < nblk && (b & 3) == wave && (b >> 2) % nsplit_cfg == split) bov = b;
    }
    bov = __builtin_amdgcn_readfirstlane(bov);
  }
  pk_cw_t Kb = Kc + (long)hh * capb * 2048 + lane * 8;
  pk_cw_t Vb = Vc + (long)hh * capb * 2048 + (lane & 15) * 32 + g * 8;
  f16x8 ka[2][4], va[2][4];
  auto load = [&](f16x8 (&kf)[4], f16x8 (&vf)[4], int b) {
#pragma unroll
    for (int f = 0; f < 4; f++) kf[f] = *(const PK_GLOBAL f16x8*)(Kb + (long)b * 2048 + f * 512);
#pragma unroll
    for (int dt = 0; dt < 4; dt++) vf[dt] = *(const PK_GLOBAL f16x8*)(Vb + (long)b * 2048 + dt * 512);
  };
  if (b0 < nblk) load(ka[0], va[0], b0);
  // q of this lane: dims g*8..+8 and 32 + g*8..+8 of the head = two runs of four tagged elements = four 16-byte
  // agent-scope loads per query tile, simply repeated until every tag matches (small enough to poll with the data itself).  Where one
  // of the wave's blocks holds rows written by this pass, those come in the same trip: the tiles that produce them are units of the same stage.
  // (In a trip of their own behind the queries the attention stage of 1500 keys takes 3.6 us instead of 2.6 at d = 512, 6.0 instead of 4.7 at 1024.)
  f16x8 qf0[QT], qf1[QT];
  f16x8 nk[4], nv[4];       // fragments of that block, valid where fromK / fromV
  int keyK[2], keyV[8];     // positions of this lane's keys in it
  bool ok = true;
  {
    const agent_buf_t qb = agent_buf(qbuf, QT * 16 * (d >> 1) * 8);
    int qo[QT];
#pragma unroll
    for (int t = 0; t < QT; t++) qo[t] = ((on[t] ? t * 16 + ql : 0) * (d >> 1) + ((hh * 64 + g * 8) >> 1)) * 8;
    const agent_buf_t kb = agent_buf(a.newK + (long)hh * (QT * 16) * 32, QT * 16 * 32 * 8), vb = agent_buf(a.newV + (long)hh * (QT * 16) * 32, QT * 16 * 32 * 8);
    int ko[2], vo[8];
    auto row_of = [&](int key) { return min(max(key - P0, 0), R - 1) * 256; };
#pragma unroll
    for (int h = 0; h < 2; h++) { keyK[h] = held(bov * 32 + h * 16 + ql); ko[h] = row_of(keyK[h]) + g * 32; }
#pragma unroll
    for (int j = 0; j < 8; j++) { keyV[j] = held(bov * 32 + (j >> 2) * 16 + g * 4 + (j & 3)); vo[j] = row_of(keyV[j]) + (ql >> 1) * 8; }
    const u64 t0 = wall_clock64();
    int it = 0;
    u32x4 qv[QT][4];
    while (true) {
      agent_again();
      unsigned diff = 0;
#pragma unroll
      for (int t = 0; t < QT; t++)
#pragma unroll
        for (int j = 0; j < 4; j++) qv[t][j] = ld_agent4(qb, qo[t] + ((j >> 1) * 16 + (j & 1) * 2) * 8);
      if (bov >= 0) {
        u32x4 kk[4][2];
        u32x2 vv[4][8];
#pragma unroll
        for (int f = 0; f < 4; f++)
#pragma unroll
          for (int j = 0; j < 2; j++) kk[f][j] = ld_agent4(kb, ko[f >> 1] + (f & 1) * 128 + j * 16);
#pragma unroll
        for (int dt = 0; dt < 4; dt++)
#pragma unroll
          for (int j = 0; j < 8; j++) vv[dt][j] = ld_agent2(vb, vo[j] + dt * 64);
#pragma unroll
        for (int f = 0; f < 4; f++) {
          diff |= (kk[f][0][1] ^ tag) | (kk[f][0][3] ^ tag) | (kk[f][1][1] ^ tag) | (kk[f][1][3] ^ tag);
          nk[f] = __builtin_bit_cast(f16x8, (u32x4{kk[f][0][0], kk[f][0][2], kk[f][1][0], kk[f][1][2]}));
        }
#pragma unroll
        for (int dt = 0; dt < 4; dt++)
#pragma unroll
          for (int j = 0; j < 8; j++) {
            diff |= vv[dt][j][1] ^ tag;
            nv[dt][j] = __builtin_bit_cast(f16_t, (unsigned short)(ql & 1 ? vv[dt][j][0] >> 16 : vv[dt][j][0] & 0xFFFFu));
          }
      }
#pragma unroll
      for (int t = 0; t < QT; t++)
#pragma unroll
        for (int j = 0; j < 4; j++) diff |= (qv[t][j][1] ^ tag) | (qv[t][j][3] ^ tag);
      if (__all(diff == 0)) break;
      if ((++it & 63) == 0 && pk_expired(a, t0, stage)) { ok = false; break; }
    }
#pragma unroll
    for (int t = 0; t < QT; t++) {
      u32x4 lo4 = u32x4{qv[t][0][0], qv[t][0][2], qv[t][1][0], qv[t][1][2]};
      u32x4 hi4 = u32x4{qv[t][2][0], qv[t][2][2], qv[t][3][0], qv[t][3][2]};
      if (!on[t]) { lo4 = u32x4{0u, 0u, 0u, 0u}; hi4 = lo4; }
      qf0[t] = __builtin_bit_cast(f16x8, lo4);
      qf1[t] = __builtin_bit_cast(f16x8, hi4);
    }
  }

  float mrun[QT], lrun[QT];
  f32x4 o[QT][4];
#pragma unroll
  for (int t = 0; t < QT; t++) {
    mrun[t] = -INFINITY;
    lrun[t] = 0.f;
#pragma unroll
    for (int dt = 0; dt < 4; dt++) o[t][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  auto attend = [&](f16x8 (&kf)[4], f16x8 (&vf)[4], int b) {
    if (b == bov) {
#pragma unroll
      for (int f = 0; f < 4; f++)
        if (keyK[f >> 1] >= P0 && keyK[f >> 1] < P0 + R) kf[f] = nk[f];
      // From this pass: positions >= P0, all of them rows of it.  A slot that this stream has not reached (position below 0) takes the
      // value too that was fetched for it, the first row's: its probability is 0, but what an earlier mesh left there may not be
      // finite, and 0 times that is NaN.
#pragma unroll
      for (int dt = 0; dt < 4; dt++)
#pragma unroll
        for (int j = 0; j < 8; j++)
          if ((unsigned)keyV[j] >= (unsigned)P0) vf[dt][j] = nv[dt][j];
    }
#pragma unroll
    for (int t = 0; t < QT; t++) {
      f32x4 sT[2];
#pragma unroll
      for (int hb = 0; hb < 2; hb++) {
        f32x4 z = f32x4{0.f, 0.f, 0.f, 0.f};
        z = __builtin_amdgcn_mfma_f32_16x16x32_f16(kf[hb * 2], qf0[t], z, 0, 0, 0);
        z = __builtin_amdgcn_mfma_f32_16x16x32_f16(kf[hb * 2 + 1], qf1[t], z, 0, 0, 0);
        sT[hb] = z;
      }
      float mx = -INFINITY;
#pragma unroll
      for (int hb = 0; hb < 2; hb++)
#pragma unroll
        for (int i = 0; i < 4; i++) {
          const int key = held(b * 32 + hb * 16 + g * 4 + i);      // absolute position
          const float v = (key <= lim[t] && key >= first[t]) ? sT[hb][i] * kScale : -INFINITY;
          sT[hb][i] = v;
          mx = fmaxf(mx, v);
        }
      mx = rows_max(mx);
      const float mnew = fmaxf(mrun[t], mx);
      const float msafe = mnew == -INFINITY ? 0.f : mnew;
      const float alpha = __builtin_amdgcn_exp2f(mrun[t] - msafe);
      mrun[t] = mnew;
      f16x8 pf;
      float psum = 0.f;
#pragma unroll
      for (int hb = 0; hb < 2; hb++)
#pragma unroll
        for (int i = 0; i < 4; i++) {
          const float p = __builtin_amdgcn_exp2f(sT[hb][i] - msafe);
          psum += p;
          pf[hb * 4 + i] = (f16_t)p;
        }
      lrun[t] = lrun[t] * alpha + psum;
#pragma unroll
      for (int dt = 0; dt < 4; dt++) {
        o[t][dt] *= alpha;
        o[t][dt] = __builtin_amdgcn_mfma_f32_16x16x32_f16(vf[dt], pf, o[t][dt], 0, 0, 0);
      }
    }
  };
  for (int b = b0; b < nblk; b += 2 * step) {
    if (b + step < nblk) load(ka[1], va[1], b + step);
    attend(ka[0], va[0], b);
    if (b + step < nblk) {
      if (b + 2 * step < nblk) load(ka[0], va[0], b + 2 * step);
      attend(ka[1], va[1], b + step);
    }
  }
#pragma unroll
  for (int t = 0; t < QT; t++) {
    const float l = rows_sum(lrun[t]);
    // (an inactive row carries a negative sum and gives 0; a row with keys whose sum is NaN or 0 gives NaN, which the pass counts)
    if (g == 0) { sh.lm[par][wave][t * 16 + ql] = lim[t] < 0 ? 0.f : mrun[t]; sh.ll[par][wave][t * 16 + ql] = lim[t] < 0 ? -1.f : l; }
#pragma unroll
    for (int dt = 0; dt < 4; dt++) *reinterpret_cast<f32x4*>(&sh.lo[par][wave][t * 16 + ql][dt * 16 + g * 4]) = o[t][dt];
  }
  if (!pk_sync(sh, ok)) return false;
  PK_MARK(3);
  // the waves' parts meet: 16 threads per row, four dims each
#pragma unroll
  for (int t = 0; t < QT; t++) {
    const int ql16 = threadIdx.x >> 4, qi = t * 16 + ql16, j = threadIdx.x & 15;
    if (qi < R) {
      float m[4], f[4];
#pragma unroll
      for (int w = 0; w < 4; w++) m[w] = sh.lm[par][w][qi];
      const float M = fmaxf(fmaxf(m[0], m[1]), fmaxf(m[2], m[3]));
      const float Ms = M == -INFINITY ? 0.f : M;
      float den = 0.f;
#pragma unroll
      for (int w = 0; w < 4; w++) {
        f[w] = __builtin_amdgcn_exp2f(m[w] - Ms);
        den += sh.ll[par][w][qi] * f[w];
      }
      if (nact == 1) {      // the only part: the row's result, four neighbouring dims (what a merge of one part would give, bit by bit)
        f32x4 num = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < 4; w++) num += *reinterpret_cast<const f32x4*>(&sh.lo[par][w][qi][4 * j]) * f[w];
        u64* at = att + (long)qi * (d >> 1) + hh * 32 + 2 * j;
        pk_st(at, den < 0.f ? pk_pack(0.f, 0.f) : pk_pack(num[0] / den, num[1] / den), tag);
        pk_st(at + 1, den < 0.f ? pk_pack(0.f, 0.f) : pk_pack(num[2] / den, num[3] / den), tag);
        continue;
      }
      u64* pt = part + (long)t * PK_PART;
#pragma unroll
      for (int k = 0; k < 4; k++) {
        const int dim = j + 16 * k;
        float num = 0.f;
#pragma unroll
        for (int w = 0; w < 4; w++) num += sh.lo[par][w][qi][dim] * f[w];
        pk_stf(pt + ql16 * 64 + dim, num, tag);
      }
      if (j < 2) pk_stf(pt + 16 * 64 + ql16 * 2 + j, j == 0 ? M : den, tag);
    }
  }
  return true;
}

// Merge of the splits of one head into the half-pair attention output: a unit takes four rows, a wave each; lane (g, j) the dims 4j .. 4j+3 of
// the splits g, g + 4, ..., all parts in one trip of 16-byte loads (PK_MAXSPLIT); no wave waits for another.  Splits and lanes are added
// in a fixed order.  (A quarter of the dims per unit, one dim per lane and 8-byte loads, 48 of them: 3.6 us from the last part to the last trip at nine rows.)
// (row0: the first of the four rows, R: rows of the level; the split count comes from the largest limit of the whole level, as in the units
// that wrote the partial results)
template <int QT, int FWT, class SH>
__device__ __forceinline__ void pk_merge_unit(const PkArgs& a, SH& sh, int maxlim, int R, int row0, int capb, int nsplit_cfg,
                                              int hh, const u64* parts, u64* att, unsigned tag, int stage) {
  const int d = pk_d<FWT>(a);
  const int nsplit = pk_parts(maxlim, capb, nsplit_cfg);
  constexpr int rec = QT * PK_PART * 8;                 // bytes of one (head, split) record: a tile per row group
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int g = lane >> 4, j = lane & 15, row = row0 + wave;
  if (row >= R) return;
  const agent_buf_t pb = agent_buf(parts + (long)hh * PK_MAXSPLIT * QT * PK_PART, nsplit * rec);      // splits that do not exist read 0
  const int tile = (row >> 4) * PK_PART * 8, r16 = row & 15;
  u32x4 ml[4], va[4], vb[4];
  const u64 t0 = wall_clock64();
  int it = 0;
  while (true) {
    agent_again();
#pragma unroll
    for (int k = 0; k < 4; k++)
      if (4 * k < nsplit) {
        const int o = (g + 4 * k) * rec + tile;
        ml[k] = ld_agent4(pb, o + (16 * 64 + r16 * 2) * 8);
        va[k] = ld_agent4(pb, o + (r16 * 64 + 4 * j) * 8);
        vb[k] = ld_agent4(pb, o + (r16 * 64 + 4 * j + 2) * 8);
      }
    unsigned diff = 0;
#pragma unroll
    for (int k = 0; k < 4; k++)
      if (4 * k < nsplit && g + 4 * k < nsplit)
        diff |= (ml[k][1] ^ tag) | (ml[k][3] ^ tag) | (va[k][1] ^ tag) | (va[k][3] ^ tag) | (vb[k][1] ^ tag) | (vb[k][3] ^ tag);
    if (__all(diff == 0)) break;
    if ((++it & 63) == 0 && pk_expired(a, t0, stage)) { sh.bad = 1; return; }
    __builtin_amdgcn_s_sleep(1);
  }
  PK_MARK(2);
  float M = -INFINITY;
#pragma unroll
  for (int k = 0; k < 4; k++) if (g + 4 * k < nsplit) M = fmaxf(M, __uint_as_float(ml[k][0]));
  M = rows_max(M);
  const float Ms = M == -INFINITY ? 0.f : M;
  float den = 0.f;
  f32x4 num = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int k = 0; k < 4; k++)
    if (g + 4 * k < nsplit) {
      const float f = __builtin_amdgcn_exp2f(__uint_as_float(ml[k][0]) - Ms);
      den += __uint_as_float(ml[k][2]) * f;
      num[0] += __uint_as_float(va[k][0]) * f; num[1] += __uint_as_float(va[k][2]) * f;
      num[2] += __uint_as_float(vb[k][0]) * f; num[3] += __uint_as_float(vb[k][2]) * f;
    }
  den = rows_sum(den);
#pragma unroll
  for (int i = 0; i < 4; i++) num[i] = rows_sum(num[i]);
  if (g < 2) {       // row g of lanes stores dims 4j + 2g, 4j + 2g + 1
    const float x = g == 0 ? num[0] : num[2], y = g == 0 ? num[1] : num[3];
    pk_st(att + (long)row * (d >> 1) + hh * 32 + 2 * j + g, den < 0.f ? pk_pack(0.f, 0.f) : pk_pack(x / den, y / den), tag);
  }
}

// ------------------------------------------------------------------------------------------
// The kernel
// ------------------------------------------------------------------------------------------
#define PK_MINE(units) for (int u = (int)((blockIdx.x + PK_NWG - (rr % PK_NWG)) % PK_NWG); u < (units) && (worked = true); u += PK_NWG)
#define PK_NEXT(units)                                                                              \
  do {                                                                                              \
    if (a.prof && worked) PK_STAMP(1 + stage);                                                      \
    worked = false;                                                                                 \
    rr += (units);                                                                                  \
    stage++;                                                                                        \
  } while (0)

template <int QT, int FWT>
__global__ __launch_bounds__(256) void k_verify_persist(PkArgs a) {
  const unsigned epoch = __builtin_amdgcn_readfirstlane((int)*a.epoch_word);
  if (*a.run_flag == 0) return;
  __shared__ PkShared<QT> sh;
  if (threadIdx.x == 0) sh.bad = 0;
  __syncthreads();
  const int RS = QT * 16, RH = QT * 8;     // rows of an exchange region (= a.RS), and half of it: the row count of a half-pair region in units of d
  const int d = pk_d<FWT>(a), H = d / 64, ff = FWT ? 4 * d : a.ff;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  unsigned rr = 0;     // round-robin origin of the current stage (same in every workgroup)
  int stage = 0, par = 0;
  // this thread's place in a GEMM tile: row of the group, column of the tile
  const int er = ((threadIdx.x & 63) >> 4) * 4 + wave, ec = threadIdx.x & 15;
  bool worked = false;
  if (a.prof && threadIdx.x == 0) atomicMin(a.prof, (u64)wall_clock64());

  // Per level and the same for all of its layers: the last visible key of this lane's query row in the
  // self-attention (its own position) and in the cross-attention, the block maxima, the first position of the pass.
  // (QT query tiles of 16 rows: tile t holds rows t*16 .. t*16+15 of the level)
  int limS[3][QT], limX[3][QT], maxS[3], maxX[3], firstP[3];
#pragma unroll
  for (int lv = 0; lv < 3; lv++) {
    const int ql = threadIdx.x & 15;
    int ms = -1, mx = -1, fp = 0x3fffffff;
#pragma unroll
    for (int t = 0; t < QT; t++) {
      const bool onl = t * 16 + ql < a.R[lv];
      limS[lv][t] = onl ? a.pos[lv][t * 16 + ql] : -1;
      limX[lv][t] = onl ? a.limx[lv][t * 16 + ql] : -1;
      ms = max(ms, limS[lv][t]);
      mx = max(mx, limX[lv][t]);
      if (limS[lv][t] >= 0) fp = min(fp, limS[lv][t]);
    }
#pragma unroll
    for (int o = 1; o < 16; o <<= 1) {
      ms = max(ms, __shfl_xor(ms, o, 64));
      mx = max(mx, __shfl_xor(mx, o, 64));
      fp = min(fp, __shfl_xor(fp, o, 64));
    }
    maxS[lv] = ms; maxX[lv] = mx; firstP[lv] = fp;
  }

  // ---- embedding: one unit per coordinate row -> hA of layer 0
  PK_MINE(a.R[0]) {
    const int r = u;
    const bool onr = a.pos[0][r] >= 0;
    const f16_t* e = a.emb + (long)a.vtok[r] * d;
    const int n = SkipCols::count(d, threadIdx.x);
    float v[FM_TR_COLS], gain[FM_TR_COLS];
#pragma unroll
    for (int k = 0; k < FM_TR_COLS; k++) {           // all loads together
      const int i = min(SkipCols::col(threadIdx.x, k), d - 1);
      v[k] = (float)e[i];
      gain[k] = ((pk_cf_t)a.layers[0].g1)[i];
    }
#pragma unroll
    for (int k = 0; k < FM_TR_COLS; k++) {           // region of layer 0, and its copy for the first norm (d is a multiple of 128)
      if (k >= n) break;
      pk_put_row(onr ? v[k] : 0.f, true, r, SkipCols::col(threadIdx.x, k), d, a.hA, a.xA, a.sA, gain[k], PK_TAG(0) + a.test_skew);
    }
  }
  PK_NEXT(a.R[0]);

  for (int st = 0; st < 5; st++) {
    for (int li = 0; li < a.count[st]; li++) {
      const int l = a.first[st] + li;
      const PkLayer& L = a.layers[l];
      const int lev = L.level, R = a.R[lev];
      const unsigned tag = PK_TAG(l);
      const int* pos = a.pos[lev];
      const int capb = a.capb[lev];
      // this layer's own regions of the exchange buffers
      u64* const hA_l = a.hA + (long)l * RS * d;
      u64* const hA_n = a.hA + (long)(l + 1) * RS * d;
      u64* const hB_l = a.hB + (long)l * RS * d;
      u64* const hC_l = a.hC + (long)l * RS * d;
      u64* const xA_l = a.xA + (long)l * RH * d;
      u64* const xA_n = a.xA + (long)(l + 1) * RH * d;
      u64* const xB_l = a.xB + (long)l * RH * d;
      u64* const xC_l = a.xC + (long)l * RH * d;
      u64* const sA_l = a.sA + (long)l * RS * (d >> 4);
      u64* const sB_l = a.sB + (long)l * RS * (d >> 4);
      u64* const sC_l = a.sC + (long)l * RS * (d >> 4);
      u64* const att_l = a.att + (long)l * RH * d;
      u64* const att2_l = a.att2 + (long)l * RH * d;
      u64* const mid_l = a.mid + (long)l * RH * ff;
      // GEMM units take the rows in groups of 16: unit = (tile, row group); a group's rows are contiguous
      // in every exchange buffer, so a unit is the one-group code on offset pointers
      const int RG = QT == 1 ? 1 : (R + 15) >> 4;      // a compile-time 1 for blocks of up to 16 tokens
      const int RQ = (R + 3) >> 2;                     // merge units: four rows of a head each
      const long hd = d >> 1, sd = d >> 4;
      // ---- QKV (norm1 on the fly, rotary, q / new K,V out, cache append)
      PK_MINE(3 * d / 16 * RG) {
        const int nt = u / RG, row0 = (u % RG) * 16, Rl = min(16, R - row0);
        float c;
        PkQkvPre pre;
        pk_qkv_prefetch(nt, d, Rl, pos + row0, a.cs[lev] + (long)row0 * 32, pre);
        if (!pk_gemm_tile<FWT, true>(a, sh, par, L.wqkv + (long)nt * (d / 32) * 512, d / 32, xA_l + row0 * hd, tag, sA_l + row0 * sd, Rl, c, stage)) return;
        pk_epi_qkv<QT, FWT>(a, L, c, nt, tag, Rl, pre, capb, row0);
      }
      PK_NEXT(3 * d / 16 * RG);
      // ---- self-attention splits
      {
        const int ns = a.nsplit[lev];
        const int P0 = firstP[lev];
        PK_MINE(H * ns) {
          // split-major: the splits that hold keys come first and spread over all workgroups
          const int hh = u % H, sp = u / H;
          if (!pk_attn_unit<QT, FWT>(a, sh, par, a.q, limS[lev], maxS[lev], R, L.Kc, L.Vc, capb, ns, hh, sp, true, P0,
                                a.partS + ((long)hh * PK_MAXSPLIT + sp) * (RS >> 4) * PK_PART, att_l, tag, stage, a.win[lev])) return;
        }
        PK_NEXT(H * ns);
        if (pk_parts(maxS[lev], capb, ns) > 1) PK_MINE(H * RQ) pk_merge_unit<QT, FWT>(a, sh, maxS[lev], R, u / H * 4, capb, ns, u % H, a.partS, att_l, tag, stage);
        PK_NEXT(H * RQ);
      }
      // ---- Wo + residual -> hB (tap: the layer input is what the draft heads of this level start from)
      PK_MINE(d / 16 * RG) {
        const int nt = u / RG, row0 = (u % RG) * 16, Rl = min(16, R - row0);
        const int n = nt * 16 + ec;
        float c, old;
        PkOld res;
        pk_res_request<FWT>(a, n, hA_l + (long)row0 * d, Rl, pos + row0, L.g2, res);
        if (!pk_gemm_tile<FWT, false>(a, sh, par, L.wo + (long)nt * (d / 32) * 512, d / 32, att_l + row0 * hd, tag, nullptr, Rl, c, stage)) return;
        if (pk_res_take<FWT>(a, n, hA_l + (long)row0 * d, tag, Rl, res, old, stage)) {
          pk_put_row(old + c, er < Rl, er, n, d, hB_l + (long)row0 * d, xB_l + row0 * hd, sB_l + row0 * sd, res.gain, tag);
          if (L.tap && er < Rl && res.p >= 0) a.tap[lev][(long)(res.p & (lev == 0 ? 31 : lev == 1 ? 15 : 7)) * d + n] = old;
        } else sh.bad = 1;
      }
      PK_NEXT(d / 16 * RG);
      // ---- cross-attention query (norm2 on the fly)
      PK_MINE(d / 16 * RG) {
        const int nt = u / RG, row0 = (u % RG) * 16, Rl = min(16, R - row0);
        float c;
        if (!pk_gemm_tile<FWT, true>(a, sh, par, L.cq + (long)nt * (d / 32) * 512, d / 32, xB_l + row0 * hd, tag, sB_l + row0 * sd, Rl, c, stage)) return;
        pk_put_half(c, er < Rl, er, nt * 16 + ec, a.q2 + row0 * hd, d >> 1, tag);
      }
      PK_NEXT(d / 16 * RG);
      // ---- cross-attention over the condition memory
      {
        const int ns = a.nsplitM;
        PK_MINE(H * ns) {
          const int hh = u / ns, sp = u % ns;
          if (!pk_attn_unit<QT, FWT>(a, sh, par, a.q2, limX[lev], maxX[lev], R, L.Km, L.Vm, a.capbM, ns, hh, sp, false, 0,
                                a.partX + ((long)hh * PK_MAXSPLIT + sp) * (RS >> 4) * PK_PART, att2_l, tag, stage, 0)) return;
        }
        PK_NEXT(H * ns);
        if (pk_parts(maxX[lev], a.capbM, ns) > 1) PK_MINE(H * RQ) pk_merge_unit<QT, FWT>(a, sh, maxX[lev], R, u / H * 4, a.capbM, ns, u % H, a.partX, att2_l, tag, stage);
        PK_NEXT(H * RQ);
      }
      // ---- cross output projection + residual -> hC
      PK_MINE(d / 16 * RG) {
        const int nt = u / RG, row0 = (u % RG) * 16, Rl = min(16, R - row0);
        const int n = nt * 16 + ec;
        float c, old;
        PkOld res;
        pk_res_request<FWT>(a, n, hB_l + (long)row0 * d, Rl, pos + row0, L.g3, res);
        if (!pk_gemm_tile<FWT, false>(a, sh, par, L.co + (long)nt * (d / 32) * 512, d / 32, att2_l + row0 * hd, tag, nullptr, Rl, c, stage)) return;
        if (pk_res_take<FWT>(a, n, hB_l + (long)row0 * d, tag, Rl, res, old, stage))
          pk_put_row(old + c, er < Rl, er, n, d, hC_l + (long)row0 * d, xC_l + row0 * hd, sC_l + row0 * sd, res.gain, tag);
        else sh.bad = 1;
      }
      PK_NEXT(d / 16 * RG);
      // ---- FFN up (norm3 on the fly, GELU)
      PK_MINE(ff / 16 * RG) {
        const int nt = u / RG, row0 = (u % RG) * 16, Rl = min(16, R - row0);
        float c;
        if (!pk_gemm_tile<FWT, true>(a, sh, par, L.w1 + (long)nt * (d / 32) * 512, d / 32, xC_l + row0 * hd, tag, sC_l + row0 * sd, Rl, c, stage)) return;
        pk_put_half(gelu_tanh_f(c), er < Rl, er, nt * 16 + ec, mid_l + (long)row0 * (ff >> 1), ff >> 1, tag);
      }
      PK_NEXT(ff / 16 * RG);
      // ---- FFN down + residual -> next layer input, or the stack output (+ its ring for later passes).
      // K = ff is four times longer than in the other GEMMs, so a tile is computed by four units, one per
      // K-quarter; quarters 1..3 hand their partial tile to quarter 0, which adds them in a fixed order.
      PK_MINE(4 * (d / 16) * RG) {
        const int uv = u / RG, rg = u % RG, row0 = rg * 16, Rl = min(16, R - row0);
        const int nt = uv >> 2, kq = uv & 3;
        const int KTq = ff / 128;                       // fragments of one K-quarter
        u64* const w2p = a.w2part + ((long)nt * RG + rg) * 3 * 256;
        const int n = nt * 16 + ec;
        float c, old;
        PkOld res;
        // the norm behind this layer: the next one's first, the output head's behind the last
        const bool out = L.last && st < 4;       // a stack output feeds a level transition, not a norm
        if (kq == 0) pk_res_request<FWT>(a, n, hC_l + (long)row0 * d, Rl, pos + row0, out ? nullptr : L.last ? (pk_cf_t)a.gf : a.layers[l + 1].g1, res);
        if (!pk_gemm_tile<FWT, false>(a, sh, par, L.w2 + ((long)nt * (ff / 32) + (long)kq * KTq) * 512, KTq,
                                      mid_l + (long)row0 * (ff >> 1) + (long)kq * (ff / 8), tag, nullptr, Rl, c, stage, ff >> 1)) return;
        if (kq > 0) {
          pk_stf(w2p + (long)(kq - 1) * 256 + threadIdx.x, c, tag);
        } else {
          // rows that do not exist wait for nothing: nobody waits for them either, and the next layer writes the same partial tiles
          unsigned pr[3];
          if (pk_fetch<3>(pr, 3, er < Rl, tag, [&](int i) { return w2p + (long)i * 256 + threadIdx.x; }, a, stage) &&
              pk_res_take<FWT>(a, n, hC_l + (long)row0 * d, tag, Rl, res, old, stage)) {
            PK_MARK(4);
#pragma unroll
            for (int k = 0; k < 3; k++) c += __uint_as_float(pr[k]);
            const float v = old + c;
            pk_put_row(v, er < Rl, er, n, d, (out ? a.hT[st] : hA_n) + (long)row0 * d, out ? nullptr : xA_n + row0 * hd,
                       a.sA + (long)(l + 1) * RS * sd + row0 * sd, res.gain, PK_TAG(l + 1));
            if (out && er < Rl && res.p >= 0) {
              float* ring = st == 0 ? a.ring_hc : st == 1 ? a.ring_hv : st == 2 ? a.ring_yf : a.ring_yv;
              ring[(long)(res.p & (st == 0 ? 31 : st == 2 ? 7 : 15)) * d + n] = v;
            }
          } else sh.bad = 1;
        }
      }
      PK_NEXT(4 * (d / 16) * RG);
    }
    // ---- level transition after stack st; everything it produces carries the tag of the next layer
    const int ln = a.first[st] + a.count[st];
    const unsigned tagn = PK_TAG(ln);
    if (st == 0 || st == 1) {
      // shorten: coarse slot k pools fine positions 3j-2..3j (this pass: stack output; older: ring; before the start: 0)
      const int fl = st, cl = st + 1;
      const float* ring = st == 0 ? a.ring_hc : a.ring_hv;
      const int rs = st == 0 ? 32 : 16;
      const int Rf_ = a.R[fl], Rc_ = a.R[cl];
      const int F0 = firstP[fl];   // first fine position of this pass
      PK_MINE(Rc_) {
        constexpr int C = FM_TR_COLS;
        const int j = firstP[cl] + u <= maxS[cl] ? firstP[cl] + u : -1;      // active rows are the first ones, positions side by side
        const int p0 = 3 * j - 2;      // positions p0 .. p0 + 2; j < 0: an inactive row, zeros
        float was[3][C], now[3][C];
#pragma unroll
        for (int q = 0; q < 3; q++)
#pragma unroll
          for (int k = 0; k < C; k++) was[q][k] = ring[(long)((p0 + q) & (rs - 1)) * d + min(PoolCols::col(threadIdx.x, k), d - 1)];
        const bool ok = pk_wait_stack<FWT, PoolCols>(a, a.hT[st], tagn, stage, Rf_, [&](int q) { return min(max(p0 + q - F0, 0), Rf_ - 1); }, now);
#pragma unroll
        for (int k = 0; k < C; k += 2) {
          const int i = PoolCols::col(threadIdx.x, k);   // two adjacent columns per thread
          float s0 = 0.f, s1 = 0.f;
#pragma unroll
          for (int q = 0; q < 3; q++) {
            const bool in = p0 + q >= F0, on = j >= 0 && p0 + q >= 0;
            s0 += !on ? 0.f : in ? now[q][k] : was[q][k];
            s1 += !on ? 0.f : in ? now[q][k + 1] : was[q][k + 1];
          }
          if (i < d) pk_st(a.pool + (long)st * 8 * d + (long)u * (d >> 1) + (i >> 1), pk_pack(s0 / 3.0f, s1 / 3.0f), tagn);
        }
        if (!ok) sh.bad = 1;
      }
      PK_NEXT(Rc_);
      PK_MINE(d / 16) {
        float c;
        const float gain = a.layers[ln].g1[u * 16 + ec];
        pk_cw_t W = (pk_cw_t)(st == 0 ? a.short_cv : a.short_vf) + (long)u * (d / 32) * 512;
        if (!pk_gemm_tile<FWT, false>(a, sh, par, W, d / 32, a.pool + (long)st * 8 * d, tagn, nullptr, Rc_, c, stage)) return;
        pk_put_row(c, er < Rc_, er, u * 16 + ec, d, a.hA + (long)ln * RS * d, a.xA + (long)ln * RH * d, a.sA + (long)ln * RS * (d >> 4), gain, tagn);
      }
      PK_NEXT(d / 16);
    } else if (st == 2 || st == 3) {
      // upsample: fine row = skip (output of the level's first half) + coarse output of slot floor(pos/3)
      const int fl = st == 2 ? 1 : 0, cl = fl + 1;
      const u64* skip = a.hT[st == 2 ? 1 : 0];
      const unsigned tag_skip = PK_TAG(a.first[st == 2 ? 1 : 0] + a.count[st == 2 ? 1 : 0]);
      const float* ring = st == 2 ? a.ring_yf : a.ring_yv;
      const int rs = st == 2 ? 8 : 16;
      const int Rf_ = a.R[fl], Rc_ = a.R[cl];
      PK_MINE(Rf_) {
        constexpr int C = FM_TR_COLS;
        const int p = firstP[fl] + u <= maxS[fl] ? firstP[fl] + u : -1;      // active rows are the first ones, positions side by side
        const int slot = p / 3 - firstP[cl];                                  // row of the coarse output, below 0: it is in the ring
        const int n = SkipCols::count(d, threadIdx.x);
        // what has been there since the level's first half leaves in front of the wait
        const agent_buf_t kb = agent_buf(skip, Rf_ * d * 8);
        u32x2 kept[C];
        float was[C], now[1][C], gain[C];
#pragma unroll
        for (int k = 0; k < C; k++) {
          const int i = min(SkipCols::col(threadIdx.x, k), d - 1);
          kept[k] = ld_agent2(kb, (u * d + i) * 8);
          was[k] = ring[(long)((max(p, 0) / 3) & (rs - 1)) * d + i];
          gain[k] = a.layers[ln].g1[i];
        }
        bool ok = pk_wait_stack<FWT, SkipCols>(a, a.hT[st], tagn, stage, Rc_, [&](int) { return min(max(slot, 0), Rc_ - 1); }, now);
#pragma unroll
        for (int k = 0; k < C; k++) {
          if (k >= n) break;
          const int i = SkipCols::col(threadIdx.x, k);
          unsigned raw[1] = {kept[k][0]};
          if (!__all(kept[k][1] == tag_skip)) ok = pk_fetch<1>(raw, 1, true, tag_skip, [&](int) { return skip + (long)u * d + i; }, a, stage) && ok;
          const float v = __uint_as_float(raw[0]) + (p < 0 ? 0.f : slot >= 0 ? now[0][k] : was[k]);
          pk_put_row(v, true, u, i, d, a.hA + (long)ln * RS * d, a.xA + (long)ln * RH * d, a.sA + (long)ln * RS * (d >> 4), gain[k], tagn);
        }
        if (!ok) sh.bad = 1;
      }
      PK_NEXT(Rf_);
    }
  }
  // ---- output head: final norm on the fly, logits to plain memory (later launches read them)
  {
    const int l = a.n_layers, R = a.R[0];
    const int NT = (a.D.V + 15) / 16, RG = QT == 1 ? 1 : (R + 15) >> 4;
    PK_MINE(NT * RG) {
      const int nt = u / RG, row0 = (u % RG) * 16, Rl = min(16, R - row0);
      float c;
      if (!pk_gemm_tile<FWT, true>(a, sh, par, (pk_cw_t)a.lm + (long)nt * (d / 32) * 512, d / 32, a.xA + (long)l * RH * d + (long)row0 * (d >> 1),
                                   PK_TAG(l), a.sA + ((long)l * RS + row0) * (d >> 4), Rl, c, stage)) return;
      const int n = nt * 16 + ec;
      if (er < Rl && n < a.D.V) a.logits[(long)(row0 + er) * a.D.V + n] = c;
    }
  }
}

// The instance of a context: two row groups or one, and the width where the compiler's knowing it measures faster than reading it from the
// arguments.  Verify pass of 20 blocks behind 4500 tokens, us, sized against general: one row group d = 256 468 / 479, 512 524 / 525 (eight
// faces token by token 30 110 / 30 560), 768 573 / 585; two row groups 512 601 / 604, 768 678 / 711.  No faster, and hence general: two row
// groups at 256 (541 / 542), and 1024, whose eight fragments a wave are what the general instance holds anyway (40 blocks behind 9000 tokens:
// 1365 / 1368, two row groups 1639 / 1636).
typedef void (*pk_kernel_t)(PkArgs);
inline pk_kernel_t pk_kernel(const PkArgs& a) {
  const int d = a.ff == 4 * a.D.d ? a.D.d : 0;
  if (a.RS == 32) return d == 512 ? k_verify_persist<2, 4> : d == 768 ? k_verify_persist<2, 6> : k_verify_persist<2, 0>;
  return d == 256 ? k_verify_persist<1, 2> : d == 512 ? k_verify_persist<1, 4> : d == 768 ? k_verify_persist<1, 6> : k_verify_persist<1, 0>;
}
