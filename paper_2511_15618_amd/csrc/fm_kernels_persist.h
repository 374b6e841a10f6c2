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
typedef PK_GLOBAL float* pk_f_t;            // rings, logits
typedef const PK_GLOBAL int* pk_ci_t;
typedef PK_GLOBAL u64* pk_x_t;              // exchange buffers
typedef float f32x2 __attribute__((ext_vector_type(2)));
// The kernel's arguments where they lie: reads of them are scalar loads, and no store of the kernel makes the compiler read them again.
#define PK_CONST const __attribute__((address_space(4)))

// The stages of a block in their order, then what stands between stacks, then the output head.
enum { PK_QKV = 0, PK_ATT, PK_MRG, PK_WO, PK_CQ, PK_XATT, PK_XMRG, PK_CO, PK_W1, PK_W2, PK_POOL, PK_SHORT, PK_UP, PK_LM };

// Pointers of a stage, laid out by the host; a workgroup holds all records in LDS (from memory, each would be a cold trip in front of the cold
// trip to what it points at).  Eight per layer: q,k,v; self-attention; self output; cross query; cross-attention; cross output; FFN up;
// FFN down; behind the layers the two shortenings and the output head.
//   GEMM: 0 weights, 1 input rows, 2 their sums of squares (null: no norm), 3 residual stream that is added, 4 output, and for rows that go on 5 their copy
//     for the norm behind them (null: none), 6 its sums of squares, 7 its gain, 8 ring (null: none).
//   q,k,v: 4 queries, 5, 6 new keys and values, 3, 8 caches, 7 rotary table.
//   attention: 0, 1 keys and values, 2 queries, 3 parts, 4 output, 5 splits and capacity in blocks, 6 sliding window (0 = none; the caches of the
//     self-attention are then rings of that capacity).
struct PkRecord { u64 p[9]; };
#define PK_RECS 8
#define PK_MAX_RECORDS (61 * PK_RECS + 3)      // layers + 2 fit the six bits of a tag

struct PkArgs {
  const PK_GLOBAL PkRecord* records;      // [n_records], readable up to whole KiB
  int n_layers, n_records;
  int first[5], count[5];
  Dims D;
  int ff;
  float eps;
  int R[3];                 // row slots per level (<= RS)
  int RS;                   // rows the exchange buffers hold per region: 16, or 32 when the coordinate level has two row groups
  int capb[3], capbM;       // cache capacity in 32-key blocks per level / of the condition memory
  int nsplit[3], nsplitM;   // launch-time split counts (fixed partition of the key axis)
  pk_ci_t pos[3];
  pk_ci_t vtok;
  pk_f_t ring[4];           // outputs of cpre, vpre, face, vpost by position
  pk_cw_t emb;
  pk_cf_t gain1[5];         // gain of the first norm of each stack
  pk_f_t logits;
  // Exchange buffers (u64 = payload | tag << 32) that the stages outside of the records name:
  pk_x_t h, x, s;           // rows in front of a layer [layers + 1][RS][d]: one region per layer, written once per launch; half(row times the gain of the
                            // norm that reads it) [layers + 1][RS][d/2], pairs; sums of squares of 16 columns of those rows [layers + 1][RS][d/16]
  pk_x_t hT[4];             // outputs of cpre, vpre, face, vpost  [RS][d]
  pk_x_t pool;              // [2][16][d/2] pooled groups before the two shortening projections (coarse rows: at most 9)
  pk_x_t newK, newV;        // [H][RS][32]
  pk_x_t w2part;            // [d/16][RS/16][3][256]: partial tiles of the K-quarters 1..3 of the FFN down projection
  const unsigned* epoch_word;  // passes so far, counted by k_verify_setup
  u64 timeout_ticks;        // bound of every wait (100 MHz wall clock)
  unsigned test_skew;       // test hook: added to the tag the embedding publishes, so that nothing downstream ever arrives
  unsigned* abort_word;     // [0] abort flag, [1] earliest stage that gave up, [2] claim, [3..8] expected tag, tag seen,
                            // stage, workgroup, thread, element of the first missing value
  const int* run_flag;
  int prof_stage;           // stage whose inner phases are timed into prof[600..]
  u64* prof;                // optional [1 + stages]: earliest start, latest completion per stage (wall clock ticks)
};
typedef PK_CONST PkArgs PkA;

// Width of the model: FWT fragments of 32 per wave in a GEMM over d, i.e. d = 128 FWT, known to the compiler for some widths (pk_kernel;
// the hidden width is then 4 d), read from the arguments for the others (FWT = 0).
template <int FWT> __device__ __forceinline__ int pk_d(PkA& a) { return FWT ? FWT * 128 : a.D.d; }

// Exchanges between the waves of a workgroup.  Two sets, used by the GEMM and attention units in turn: a unit writes its set, passes its one
// barrier and reads; who writes the same set two units later has passed the barrier between, so all have read.
template <int QT>
struct PkShared {
  float red[2][4][4][64];
  float ssq[2][4][16];
  __align__(16) float lo[2][4][16 * QT][68];
  float lm[2][4][16 * QT], ll[2][4][16 * QT];
  int bad;                  // raised by a wave whose wait gave up
  __align__(16) PkRecord rec[(PK_MAX_RECORDS * sizeof(PkRecord) + 1023) / 1024 * 1024 / sizeof(PkRecord) + 1];
};

// Has a wave of this workgroup given up?  What a unit publishes after that is noise under a valid tag: the abort word is up, so the pass accepts and
// commits nothing, and what it wrote to caches and rings belongs to positions that are not committed.
template <class SH> __device__ __forceinline__ bool pk_bad(const SH& sh) { return __builtin_amdgcn_readfirstlane(sh.bad) != 0; }
// a record, lane k has pointer k; and one of its pointers, uniform
template <class SH> __device__ __forceinline__ u64 pk_record(const SH& sh, int i) { return sh.rec[i].p[min((int)(threadIdx.x & 63), 8)]; }
template <class P> __device__ __forceinline__ P pk_ptr(u64 rec, int k) {
  const unsigned lo = __builtin_amdgcn_readlane((int)(unsigned)rec, k), hi = __builtin_amdgcn_readlane((int)(unsigned)(rec >> 32), k);
  return (P)((u64)hi << 32 | lo);
}
// The thread's number, new to the compiler at each call: what a unit derives from it (offsets, row and column of a tile) is not computed ahead
// of the loop over the stages and kept for all units at once.
__device__ __forceinline__ int pk_tid() {
  int t = threadIdx.x;
  asm volatile("" : "+v"(t));
  return t;
}

// Barrier of a unit.  Whether a wave has given up is looked at behind the unit's results (pk_bad): an LDS trip that nobody waits for.  (In front of
// them: steps of 595 us at d = 512 and 1484 at d = 1024 instead of 590 and 1463.)
template <class SH>
__device__ __forceinline__ void pk_sync(SH& sh, bool good) {
  if (!good) sh.bad = 1;
  __syncthreads();
}

__device__ __forceinline__ u64 pk_ld(pk_x_t p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ __forceinline__ void pk_st(pk_x_t p, unsigned payload, unsigned tag) {
  __hip_atomic_store(p, ((u64)tag << 32) | payload, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void pk_stf(pk_x_t p, float v, unsigned tag) { pk_st(p, __float_as_uint(v), tag); }
__device__ __forceinline__ agent_buf_t pk_buf(pk_x_t p, int bytes) { return agent_buf((const void*)p, bytes); }
__device__ __forceinline__ unsigned pk_pack(float lo, float hi) {
  const f16_t a = (f16_t)lo, b = (f16_t)hi;
  return (unsigned)__builtin_bit_cast(unsigned short, a) | ((unsigned)__builtin_bit_cast(unsigned short, b) << 16);
}
__device__ __forceinline__ bool pk_expired(PkA& a, u64 t0, int stage) {
  // every waiter that gives up records its stage; the smallest one is where the chain broke
  if (__builtin_amdgcn_readfirstlane((int)__hip_atomic_load(a.abort_word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))) {
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
__device__ __forceinline__ bool pk_fetch(unsigned (&out)[N], int n, bool active, unsigned tag, F addr, PkA& a, int stage) {
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
__device__ __forceinline__ bool pk_wait_stack(PkA& a, pk_x_t hT, unsigned tag, int stage, int rows, ROW row, float (&got)[OWN][FM_TR_COLS]) {
  const int d = pk_d<FWT>(a);
  const int n = COLS::count(d, threadIdx.x);
  const agent_buf_t hb = pk_buf(hT, rows * d * 8);
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
// A is a half-pair exchange buffer [16][K/2].  sq not null: its rows are half(x * gain), written so by the producers of the residual stream
// together with the sums of squares of every 16 columns, sq[row][K/16]; the row factor 1/rms goes onto the result.
// (One wave doing the whole epilogue, and gain and sums computed here: steps of 707 us at d = 512 and 1692 us at d = 1024, against 644 and
// 1526 with the merge below.)
// Every wave takes the MFMA A-fragments of its K-quarter straight from the exchange buffer: lane (r, g) of
// fragment f needs the 8 consecutive values k0 = f*32 + g*8 .. +8 of row r, which are 32 contiguous bytes of
// tagged half pairs, i.e. two 16-byte agent-scope loads.  No LDS staging, no barrier before the multiplication;
// the tags are checked per lane and the whole set is re-read until complete.
// ------------------------------------------------------------------------------------------
// Weights, keys and values: with one row group a unit is the only one that reads them in the launch, and takes them as non-temporal loads.  Two row groups
// read every weight tile twice, on two dies.  Steps without / with the hint, us: d = 512 580 / 564, d = 256 515 / 508, d = 768 664 / 658, d = 1024 1451 / 1441;
// with two groups d = 512 681 / 677, d = 768 809 / 812, d = 1024 1705 / 1716 (for keys and values alone 1702 / 1705).
template <bool ONCE>
__device__ __forceinline__ f16x8 pk_once(pk_cw_t p) {
  if constexpr (ONCE) return __builtin_nontemporal_load((const PK_GLOBAL f16x8*)p);
  return *(const PK_GLOBAL f16x8*)p;
}
template <int FWT> struct PkWeights { f16x8 f[FWT ? FWT : 8]; };      // a wave's fragments of a tile
template <int FWT, bool ONCE>
__device__ __forceinline__ void pk_weights(PkWeights<FWT>& w, pk_cw_t Wt, int KT) {
  const int tid = pk_tid(), wave = __builtin_amdgcn_readfirstlane(tid >> 6), FW = FWT ? FWT : KT >> 2;
  const pk_cw_t p = Wt + (long)wave * FW * 512;
#pragma unroll
  for (int f = 0; f < (FWT ? FWT : 8); f++) {
    const int o = (f * 64 + (tid & 63)) * 8;
    if constexpr (FWT > 0) w.f[f] = pk_once<ONCE>(p + o);
    else w.f[f] = __builtin_bit_cast(f16x8, __builtin_amdgcn_raw_buffer_load_b128(agent_buf((const void*)p, FW * 1024), o * 2, 0, ONCE ? 2 : 0));      // fragments past the last are zeros; 2: non-temporal
  }
}
template <int FWT, class SH>
__device__ __forceinline__ void pk_gemm_tile(PkA& a, SH& sh, int& par, const PkWeights<FWT>& wt, int KT, pk_x_t A, int lda,
                                             unsigned tagA, pk_x_t sq, int R, float& result, int stage) {
  constexpr int NL = 2;       // 16-byte loads per fragment and lane
  constexpr int EF = 16;      // tagged elements (half pairs) per fragment row
  const bool norm = sq != nullptr;
  const int tid = pk_tid(), wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int r = lane & 15, g = lane >> 4;
  const bool on = r < R;
  constexpr int NF = FWT ? FWT : 8;
  const int FW = FWT ? FWT : KT >> 2;      // fragments per wave (host guarantees KT % 4 == 0, KT <= 32)
  const int K = FW * 128;
  par ^= 1;
  f32x4 acc[2] = {f32x4{0.f, 0.f, 0.f, 0.f}, f32x4{0.f, 0.f, 0.f, 0.f}};
  // this wave's part of the rows: element (wave*FW + f)*EF + g*(EF/4) of row r is where fragment f starts; rows past the last lie outside the
  // buffer and read 0 (a branch around every load instead: step of d = 1024 1810 -> 1907 us, d = 512 761 -> 805)
  const agent_buf_t Ab = pk_buf(A, ((R - 1) * lda + FW * 4 * EF) * 8);
  const int mine = on ? (r * lda + (wave * FW) * EF + g * (EF / 4)) * 8 : 1 << 30;
  // sums of squares of the columns of this K-quarter: pair p of 16-column sums belongs to fragment p, lane (r, g) takes p = g and g + 4
  const agent_buf_t Sb = pk_buf(norm ? sq : A, norm ? R * FW * 8 * 8 : 0);      // no norm: nothing to read, zeros that nobody looks at
  const bool son[2] = {norm && on && g < FW, norm && on && g + 4 < FW};
  int so[2];
#pragma unroll
  for (int j = 0; j < 2; j++) so[j] = son[j] ? ((r * 4 + wave) * FW + g + 4 * j) * 16 : 1 << 30;
  const u64 t0 = wall_clock64();
  int it = 0;
  bool good = true;
  // The full fragment read is its own validity check, so a unit whose input is already there pays one round trip.
  // When a read comes back incomplete the wave falls back to watching one element per lane (lane l: fragment l/8, its
  // first or second half - a producer tile owns half a fragment row - in a row of wave l%4 of that tile) and reads the
  // fragments again once those show the tag: waiting costs the memory system 64 small loads per round, not 32 KiB.  Which of a wave's rows differs
  // between workgroups, so that not all look at the same lines.  (Steps of d = 512 and 1024 in us: 583 and 1452; the last four rows for all 588 and
  // 1456; reading all again instead 658 and 1516; the sums of squares or flags of the tiles, a few lines that all waiting waves share, 715 and 1557.)
  const int fs_ = min(lane >> 3, FW - 1), hs_ = (lane >> 2) & 1, wr_ = (lane & 3) + 4 * (int)(blockIdx.x & 3), rs_ = min(wr_ < R ? wr_ : lane & 3, R - 1);
  const pk_x_t watched = A + (long)(wave * FW) * EF + (long)rs_ * lda + fs_ * EF + hs_ * (EF / 2);
  const float eps = a.eps;
  PK_MARK(1);
  u32x4 v[NF * NL], sv[2];
  while (good) {
    agent_again();
#pragma unroll
    for (int f = 0; f < NF; f++)
#pragma unroll
      for (int j = 0; j < NL; j++) v[f * NL + j] = ld_agent4(Ab, f < FW ? mine + (f * EF + 2 * j) * 8 : 1 << 30);
    sv[0] = ld_agent4(Sb, so[0]);
    if (NF > 4) sv[1] = ld_agent4(Sb, so[1]);
    unsigned diff = 0;
#pragma unroll
    for (int f = 0; f < NF; f++)
      if (f < FW)
#pragma unroll
        for (int j = 0; j < NL; j++) diff |= (v[f * NL + j][1] ^ tagA) | (v[f * NL + j][3] ^ tagA);
    if (son[0]) diff |= (sv[0][1] ^ tagA) | (sv[0][3] ^ tagA);
    if (NF > 4 && son[1]) diff |= (sv[1][1] ^ tagA) | (sv[1][3] ^ tagA);
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
    const u32x4 pk = {v[2 * f][0], v[2 * f][2], v[2 * f + 1][0], v[2 * f + 1][2]};
    acc[f & 1] = __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8, pk), wt.f[f], acc[f & 1], 0, 0, 0);
  }
  if (norm) {       // what lies outside the buffer has read 0
    float ss = __uint_as_float(sv[0][0]) + __uint_as_float(sv[0][2]);
    if (NF > 4) ss += __uint_as_float(sv[1][0]) + __uint_as_float(sv[1][2]);
    ss = rows_sum(ss);
    if (g == 0) sh.ssq[par][wave][r] = ss;
  }
  acc[0] += acc[1];
#pragma unroll
  for (int i = 0; i < 4; i++) sh.red[par][wave][i][lane] = acc[0][i];
  pk_sync(sh, good);
  PK_MARK(3);
  const int row = g * 4 + wave;
  float p[4], q[4];
#pragma unroll
  for (int k = 0; k < 4; k++) { p[k] = sh.red[par][k][wave][lane]; q[k] = sh.ssq[par][k][row]; }      // one trip to LDS
  result = p[0] + p[1] + p[2] + p[3];
  if (norm) result *= 1.0f / sqrtf((q[0] + q[1] + q[2] + q[3]) / (float)K + eps);
}

// Epilogues: a thread has row g*4 + wave (wave, lane as above) and column n = nt*16 + lane%16 of the tile.

// One value of a row of the residual stream: the value, half(value * gain of the norm that reads it) and, per 16 columns, the sum of squares.
// x null: no norm reads this row.
__device__ __forceinline__ void pk_put_row(float v, bool on, int row, int n, int d, pk_x_t h, pk_x_t x, pk_x_t sq, float gain, unsigned tag) {
  const float xg = v * gain, w = lane_xor1(xg), ss = row16_sum(v * v);
  if (!on) return;
  if (x) {
    if ((n & 1) == 0) pk_st(x + (long)row * (d >> 1) + (n >> 1), pk_pack(xg, w), tag);
    if ((n & 15) == 0) pk_stf(sq + (long)row * (d >> 4) + (n >> 4), ss, tag);
  }
  pk_stf(h + (long)row * d + n, v, tag);
}

// dst[row][n/2] = (c[n], c[n+1]) as halves
__device__ __forceinline__ void pk_put_half(float v, bool on, int row, int n, pk_x_t dst, int ld2, unsigned tag) {
  const float w = lane_xor1(v);
  if (on && (n & 1) == 0) pk_st(dst + (long)row * ld2 + (n >> 1), pk_pack(v, w), tag);
}

// QKV epilogue.  Tiles of the q and k parts hold 8 rotary pairs: columns 0..7 = dims qd*8.., columns
// 8..15 = the same dims + 32.  q -> exchange buffer; k, v -> exchange buffers and cache (for later passes).  t: rotary (cos, sin) of the
// thread's pair in its row, p: position of that row.
__device__ __forceinline__ void pk_epi_qkv(pk_x_t to, pk_w_t cache, float v, int part, int cp, unsigned tag, bool on, f32x2 t, int p, int capb, int row, int d) {
  const int lane = pk_tid() & 63, col = lane & 15;
  const int hh = cp >> 6, qd = (cp & 63) >> 4;
  int dim = qd * 16 + col;
  if (part < 2) {
    const float o = lane_xor8(v);
    v = col < 8 ? v * t[0] - o * t[1] : v * t[0] + o * t[1];
    dim = (col < 8 ? 0 : 32) + qd * 8 + (col & 7);
  }
  const float w = lane_xor1(v);       // neighbour dim (dim ^ 1 sits in lane ^ 1 in every layout above)
  if (!on) return;
  if ((lane & 1) == 0) pk_st(to + (long)row * (part == 0 ? d >> 1 : 32) + (dim >> 1), pk_pack(v, w), tag);
  if (part > 0) {
    const int ps = p % (capb * 32);      // the cache is a ring when a window is set
    cache[(long)hh * capb * 2048 + (part == 1 ? kblk_off(ps, dim) : vblk_off(ps, dim))] = (f16_t)v;
  }
}

__device__ __forceinline__ int pk_active(int nblk, int ns) { return max(1, min(ns, (nblk + 3) >> 2)); }      // splits that hold visible keys

// ------------------------------------------------------------------------------------------
// Attention over one split of the keys of one head (flash-decoding), same arithmetic and deal as k_dec_attn: block b of 32 keys
// belongs to wave b % 4 of split (b / 4) % ns, which is balanced at every length and does not depend on it.  QT tiles of
// 16 query rows share every K/V block that is loaded.  The first K/V block of a wave is requested before the wait for
// the queries, the next one behind it.  Keys of this pass (positions >= P0) are taken from the
// exchange buffers, older keys from the cache.  R rows, positions P0 ..; maxlim: the last key that one of them sees.
// Partial results: tile t of (head, split) at part + t * PK_PART.  Where one split holds all visible keys (contexts of up to 128) there is nothing
// to merge: its unit writes the attention output, and the merge stage, an exchange of 1.1 to 2 us, is left
// out (eight faces token by token at d = 512, with the trips above: 29.9 -> 26.3 ms).
// ------------------------------------------------------------------------------------------
template <int QT, int FWT, class SH>
__device__ __forceinline__ void pk_attn_unit(PkA& a, SH& sh, int& par, u64 rec, int P0, int R, int maxlim, int nact, int hh, int split,
                                             bool self, unsigned tag, int stage, int d) {
  const pk_cw_t Kc = pk_ptr<pk_cw_t>(rec, 0), Vc = pk_ptr<pk_cw_t>(rec, 1);
  const u64 sizes = pk_ptr<u64>(rec, 5);
  const int nsplit_cfg = (int)(unsigned)sizes, capb = (int)(sizes >> 32), window = (int)(unsigned)pk_ptr<u64>(rec, 6);
  const pk_x_t qbuf = pk_ptr<pk_x_t>(rec, 2), part = pk_ptr<pk_x_t>(rec, 3) + ((long)hh * PK_MAXSPLIT + split) * QT * PK_PART, att = pk_ptr<pk_x_t>(rec, 4);
  const int tid = pk_tid(), wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int g = lane >> 4, ql = lane & 15;
  const float kScale = 0.125f * 1.4426950408889634f;
  // With a window the cache is a ring of capb blocks (a multiple of four): position p lives in slot p mod (32 capb);
  // seen from the newest visible position, slot j holds lapbase + j if that is <= maxlim, else the position one
  // lap earlier.  Without a window lapbase = 0 and nothing wraps.
  const int nblk = min((maxlim + 32) >> 5, capb);
  const int ringn = capb * 32;
  const int lapbase = max(maxlim, 0) / ringn * ringn;
  auto held = [&](int slot) { const int k = lapbase + slot; return k > maxlim ? k - ringn : k; };
  bool on[QT];
  int lim[QT], first[QT];      // keys that the lane's row of tile t sees: its own position is the last one, or all of the memory; -1: no row
#pragma unroll
  for (int t = 0; t < QT; t++) {
    on[t] = t * 16 + ql < R;
    lim[t] = !on[t] ? -1 : self ? P0 + t * 16 + ql : maxlim;
    first[t] = window > 0 ? max(lim[t] - window + 1, 0) : 0;
  }
  par ^= 1;
  const int b0 = split * 4 + wave, step = nsplit_cfg * 4;     // this wave's blocks: b0, b0 + step, ...

  // The block of this wave, if any, that holds rows written by this pass.  K fragment f = (hb, dh) holds key b*32 + hb*16 + lane%16, dims
  // dh*32 + g*8..+8 (4 elements); V fragment dt holds dim dt*16 + lane%16 and the 8 slots g*8 + j <-> key b*32 + (j/4)*16 + g*4 + j%4.
  int bov = -1;
  if (self) {
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
    for (int f = 0; f < 4; f++) kf[f] = pk_once<QT == 1>(Kb + (long)b * 2048 + f * 512);
#pragma unroll
    for (int dt = 0; dt < 4; dt++) vf[dt] = pk_once<QT == 1>(Vb + (long)b * 2048 + dt * 512);
  };
  if (b0 < nblk) load(ka[0], va[0], b0);
  // q of this lane: dims g*8..+8 and 32 + g*8..+8 of the head = two runs of four tagged elements = four 16-byte
  // agent-scope loads per query tile, simply repeated until every tag matches (small enough to poll with the data itself).  Where one
  // of the wave's blocks holds rows written by this pass, those come in the same trip: the tiles that produce them are units of the same stage.
  // (In a trip of their own behind the queries the attention stage of 1500 keys takes 3.6 us instead of 2.6 at d = 512, 6.0 instead of 4.7 at 1024.)
  f16x8 qf0[QT], qf1[QT];
  f16x8 nk[4], nv[4];       // fragments of that block, in use where the key's position is one of this pass
  int keyK[2], keyV[8];     // positions of this lane's keys in it
  bool ok = true;
  {
    const agent_buf_t qb = pk_buf(qbuf, QT * 16 * (d >> 1) * 8);
    int qo[QT];
#pragma unroll
    for (int t = 0; t < QT; t++) qo[t] = ((on[t] ? t * 16 + ql : 0) * (d >> 1) + ((hh * 64 + g * 8) >> 1)) * 8;
    const agent_buf_t kb = pk_buf(a.newK + (long)hh * (QT * 16) * 32, QT * 16 * 32 * 8), vb = pk_buf(a.newV + (long)hh * (QT * 16) * 32, QT * 16 * 32 * 8);
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
  pk_sync(sh, ok);
  PK_MARK(3);
  // the waves' parts meet: 16 threads per row, four dims each
#pragma unroll
  for (int t = 0; t < QT; t++) {
    const int ql16 = tid >> 4, qi = t * 16 + ql16, j = tid & 15;
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
        pk_x_t at = att + (long)qi * (d >> 1) + hh * 32 + 2 * j;
        pk_st(at, den < 0.f ? pk_pack(0.f, 0.f) : pk_pack(num[0] / den, num[1] / den), tag);
        pk_st(at + 1, den < 0.f ? pk_pack(0.f, 0.f) : pk_pack(num[2] / den, num[3] / den), tag);
        continue;
      }
      pk_x_t pt = part + (long)t * PK_PART;
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
}

// Merge of the splits of one head into the half-pair attention output: a unit takes four rows, a wave each; lane (g, j) the dims 4j .. 4j+3 of
// the splits g, g + 4, ..., all parts in one trip of 16-byte loads (PK_MAXSPLIT); no wave waits for another.  Splits and lanes are added
// in a fixed order.  (A quarter of the dims per unit, one dim per lane and 8-byte loads, 48 of them: 3.6 us from the last part to the last trip at nine rows.)
// (row0: the first of the four rows, R: rows of the level)
template <int QT, class SH>
__device__ __forceinline__ void pk_merge_unit(PkA& a, SH& sh, int nsplit, int R, int row0, int hh, pk_x_t parts, pk_x_t att, unsigned tag, int stage, int d) {
  constexpr int rec = QT * PK_PART * 8;                 // bytes of one (head, split) record: a tile per row group
  const int tid = pk_tid(), wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
  const int g = lane >> 4, j = lane & 15, row = row0 + wave;
  if (row >= R) return;
  const agent_buf_t pb = pk_buf(parts + (long)hh * PK_MAXSPLIT * QT * PK_PART, nsplit * rec);      // splits that do not exist read 0
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

// One loop over the stages, one instance each of the GEMM, attention and merge code: what tells the stages apart are scalars and, per stage, a record of
// pointers that the host has laid out and the workgroup holds in LDS.  (With code of its own for every stage of a block an instance was 56 to 88 KB, where two compute
// units keep 64 KB of instructions, and held the offsets of all stages at once, 173 to 308 scalars of them outside of their registers, against 27 to 40 KB and 82 to 180: a
// step of d = 512 took 625 us, of d = 1024 1483, against 595 and 1471.  Pointers that are worked out from the arguments in front of each unit: 31 and 182 us more.)
// Only rows that exist take part.  A level without a row in this pass (a block that begins no vertex, no face) is left out with all its
// stacks: the finer level then takes the coarse outputs of earlier passes from the ring.  (Eight faces token by token at d = 512, where the
// vertex level has a row in every third pass and the face level in every ninth: 26.4 -> 11.5 ms, with the loop.)
template <int QT, int FWT>
__global__ __launch_bounds__(256) void k_verify_persist(PkArgs) {
  PkA& a = *(PkA*)__builtin_amdgcn_kernarg_segment_ptr();
  __shared__ PkShared<QT> sh;
  const unsigned epoch = __builtin_amdgcn_readfirstlane((int)*a.epoch_word);
  if (*a.run_flag == 0) return;
  if (threadIdx.x == 0) sh.bad = 0;
  {   // the records go straight to LDS; the barrier behind the embedding waits for them
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), bytes = a.n_records * (int)sizeof(PkRecord);
    for (int o = wave * 1024; o < bytes; o += 4096)
      __builtin_amdgcn_global_load_lds((const PK_GLOBAL void*)((const PK_GLOBAL char*)a.records + o + (threadIdx.x & 63) * 16),
                                       (__attribute__((address_space(3))) void*)((char*)sh.rec + o), 16, 0, 0);
  }
  constexpr int RS = QT * 16, RH = QT * 8;     // rows of an exchange region (= a.RS), and half of it: the row count of a half-pair region in units of d
  const int d = pk_d<FWT>(a), H = d >> 6, ff = FWT ? 4 * d : a.ff;
  const unsigned invH = (65535u + H) / H;      // u / H = u * invH >> 16 for the unit numbers of an attention stage (below 65536 / 16)
  unsigned rr = 0;         // round-robin origin of the current stage (same in every workgroup)
  int stage = 0, par = 0;
  bool worked = false;
  if (a.prof && threadIdx.x == 0) atomicMin(a.prof, (u64)wall_clock64());
  // per level: rows of this pass (positions p0 .. p0 + nr - 1) and splits of the self-attention that hold keys; splits of the cross-attention
  int p0[3], nr[3], act[3];
  auto of = [](const int (&v)[3], int lev) { return lev == 0 ? v[0] : lev == 1 ? v[1] : v[2]; };
#pragma unroll
  for (int lv = 0; lv < 3; lv++) {
    const int lane = threadIdx.x & 63, p = lane < a.R[lv] ? a.pos[lv][lane] : -1;       // active rows are the first ones, positions side by side
    nr[lv] = __popcll(__ballot(p >= 0));
    p0[lv] = nr[lv] ? __builtin_amdgcn_readfirstlane(p) : 0x3fffffff;
    act[lv] = nr[lv] ? pk_active(min((p0[lv] + nr[lv] + 31) >> 5, a.capb[lv]), a.nsplit[lv]) : 0;
  }
  const int actX = pk_active(a.capbM, a.nsplitM);
  // logits of rows that the block does not reach: zeros
  for (long i = (long)nr[0] * a.D.V + blockIdx.x * 256 + threadIdx.x; i < (long)a.R[0] * a.D.V; i += PK_NWG * 256) a.logits[i] = 0.f;
  if (nr[0] == 0) return;

  // ---- embedding: one unit per coordinate row -> residual stream of layer 0
  PK_MINE(nr[0]) {
    const int r = u;
    const pk_cw_t e = a.emb + (long)a.vtok[r] * d;
    const pk_cf_t g1 = a.gain1[0];
    const int n = SkipCols::count(d, threadIdx.x);
    float v[FM_TR_COLS], gain[FM_TR_COLS];
#pragma unroll
    for (int k = 0; k < FM_TR_COLS; k++) {           // all loads together
      const int i = min(SkipCols::col(threadIdx.x, k), d - 1);
      v[k] = (float)e[i];
      gain[k] = g1[i];
    }
#pragma unroll
    for (int k = 0; k < FM_TR_COLS; k++) {           // region of layer 0, and its copy for the first norm (d is a multiple of 128)
      if (k >= n) break;
      pk_put_row(v[k], true, r, SkipCols::col(threadIdx.x, k), d, a.h, a.x, a.s, gain[k], PK_TAG(0) + a.test_skew);
    }
  }
  PK_NEXT(nr[0]);
  __builtin_amdgcn_s_waitcnt(0x0F70);          // vmcnt(0): the records
  __syncthreads();

  // st: stack, l: layer (behind the last layer of a stack, the first one of the next), op: stage
  int st = 0, l = 0, end = a.first[1], op = PK_QKV;
  while (true) {
    const int lev = op == PK_SHORT ? st + 1 : st <= 2 ? st : 4 - st;
    const int R = of(nr, lev), P0 = of(p0, lev);
    const unsigned tag = PK_TAG(l);
    if (op == PK_ATT || op == PK_XATT) {
      // ---- attention: a unit per split that holds keys and head
      const bool self = op == PK_ATT;
      const int nact = self ? of(act, lev) : actX;
      PK_MINE(H * nact) {
        const int sp = u * invH >> 16, hh = u - sp * H;
        const u64 rec = pk_record(sh, l * PK_RECS + (self ? 1 : 4));
        pk_attn_unit<QT, FWT>(a, sh, par, rec, P0, R, self ? P0 + R - 1 : a.D.M - 1, nact, hh, sp, self, tag, stage, d);
        if (pk_bad(sh)) return;
      }
      PK_NEXT(H * nact);
    } else if (op == PK_MRG || op == PK_XMRG) {
      // ---- merge of the splits, where there are several
      const bool self = op == PK_MRG;
      const int nact = self ? of(act, lev) : actX, units = nact > 1 ? H * ((R + 3) >> 2) : 0;
      PK_MINE(units) {
        const int q = u * invH >> 16, hh = u - q * H;
        const u64 rec = pk_record(sh, l * PK_RECS + (self ? 1 : 4));
        pk_merge_unit<QT>(a, sh, nact, R, q * 4, hh, pk_ptr<pk_x_t>(rec, 3), pk_ptr<pk_x_t>(rec, 4), tag, stage, d);
      }
      PK_NEXT(units);
    } else if (op == PK_POOL) {
      // ---- shorten: coarse row of position j pools fine positions 3j-2..3j (this pass: stack output; older: ring; before the start: 0)
      const int cl = st + 1, Rc_ = of(nr, cl), rs = st == 0 ? 32 : 16;
      PK_MINE(Rc_) {
        constexpr int C = FM_TR_COLS;
        const pk_f_t ring = a.ring[st];
        const int j = of(p0, cl) + u, q0 = 3 * j - 2;
        float was[3][C], now[3][C];
#pragma unroll
        for (int q = 0; q < 3; q++)
#pragma unroll
          for (int k = 0; k < C; k++) was[q][k] = ring[(long)((q0 + q) & (rs - 1)) * d + min(PoolCols::col(threadIdx.x, k), d - 1)];
        const bool ok = pk_wait_stack<FWT, PoolCols>(a, a.hT[st], tag, stage, R, [&](int q) { return min(max(q0 + q - P0, 0), R - 1); }, now);
#pragma unroll
        for (int k = 0; k < C; k += 2) {
          const int i = PoolCols::col(threadIdx.x, k);   // two adjacent columns per thread
          float s0 = 0.f, s1 = 0.f;
#pragma unroll
          for (int q = 0; q < 3; q++) {
            const bool in = q0 + q >= P0, on = q0 + q >= 0;
            s0 += !on ? 0.f : in ? now[q][k] : was[q][k];
            s1 += !on ? 0.f : in ? now[q][k + 1] : was[q][k + 1];
          }
          if (i < d) pk_st(a.pool + (long)st * 8 * d + (long)u * (d >> 1) + (i >> 1), pk_pack(s0 / 3.0f, s1 / 3.0f), tag);
        }
        if (!ok) sh.bad = 1;
      }
      PK_NEXT(Rc_);
    } else if (op == PK_UP) {
      // ---- upsample onto level fl: skip (output of the level's first half) + coarse output of position floor(pos/3), of this pass or from the
      // ring.  st is the stack that ran last: the coarse level's, or, where that one has no row, the first half itself.
      const int fl = st >= 2 ? 3 - st : st, cl = fl + 1, Rf_ = of(nr, fl), ln = a.first[4 - fl];
      PK_MINE(Rf_) {
        constexpr int C = FM_TR_COLS;
        const pk_x_t skip = a.hT[fl];
        const pk_f_t ring = a.ring[3 - fl];
        const pk_cf_t g1 = a.gain1[4 - fl];
        const unsigned tag_skip = PK_TAG(a.first[fl] + a.count[fl]), tagn = PK_TAG(ln);
        const int p = of(p0, fl) + u, rs = fl == 1 ? 8 : 16;
        const int slot = p / 3 - of(p0, cl);                                  // row of the coarse output, below 0: it is in the ring
        const int n = SkipCols::count(d, threadIdx.x);
        // what has been there since the level's first half leaves in front of the wait
        const agent_buf_t kb = pk_buf(skip, Rf_ * d * 8);
        u32x2 kept[C];
        float was[C], now[1][C], gain[C];
#pragma unroll
        for (int k = 0; k < C; k++) {
          const int i = min(SkipCols::col(threadIdx.x, k), d - 1);
          kept[k] = ld_agent2(kb, (u * d + i) * 8);
          was[k] = ring[(long)((p / 3) & (rs - 1)) * d + i];
          gain[k] = g1[i];
        }
        bool ok = pk_wait_stack<FWT, SkipCols>(a, a.hT[st], PK_TAG(a.first[st] + a.count[st]), stage, R, [&](int) { return min(max(slot, 0), R - 1); }, now);
#pragma unroll
        for (int k = 0; k < C; k++) {
          if (k >= n) break;
          const int i = SkipCols::col(threadIdx.x, k);
          unsigned raw[1] = {kept[k][0]};
          if (!__all(kept[k][1] == tag_skip)) ok = pk_fetch<1>(raw, 1, true, tag_skip, [&](int) { return skip + (long)u * d + i; }, a, stage) && ok;
          const float v = __uint_as_float(raw[0]) + (slot >= 0 ? now[0][k] : was[k]);
          pk_put_row(v, true, u, i, d, a.h + (long)ln * RS * d, a.x + (long)ln * RH * d, a.s + (long)ln * RS * (d >> 4), gain[k], tagn);
        }
        if (!ok) sh.bad = 1;
      }
      PK_NEXT(Rf_);
      st = 4 - fl;
      l = ln;
      end = l + a.count[st];
    } else {
      // ---- GEMM.  gi: 0 q,k,v; 1 self output; 2 cross query; 3 cross output; 4 FFN up; 5 FFN down; 6 shortening; 7 output head.  Of 0 to 5 the even
      // ones read a norm's rows, the odd ones add to the residual stream.  Rows go in groups of 16: unit = (tile, row group), a group's rows
      // are contiguous in every exchange buffer.
      // FFN down: K = ff is four times longer than in the other GEMMs, so a tile is computed by four units, one per K-quarter; quarters 1..3 hand
      // their partial tile to quarter 0, which adds them in a fixed order.
      const int gi = op == PK_QKV ? 0 : op <= PK_CQ ? op - 2 : op <= PK_W2 ? op - 4 : op == PK_SHORT ? 6 : 7;
      const bool down = gi == 5, goes_on = gi == 1 || gi == 3 || gi >= 5 && gi <= 6;
      const int NT = gi == 7 ? (a.D.V + 15) >> 4 : gi == 0 ? 3 * (d >> 4) : gi == 4 ? ff >> 4 : down ? d >> 2 : d >> 4;
      const int rgs = QT == 1 || gi == 6 || R <= 16 ? 0 : 1;        // log2 of the row groups
      PK_MINE(NT << rgs) {
        const u64 rec = pk_record(sh, gi < 6 ? l * PK_RECS + gi + (gi > 0) + (gi > 2) : a.n_layers * PK_RECS + (gi == 6 ? st : 2));
        const int row0 = (u & rgs) * 16, ut = u >> rgs, nt = down ? ut >> 2 : ut, kq = down ? ut & 3 : 0, Rl = min(16, R - row0);
        const int KT = down ? ff >> 7 : d >> 5, lda = down ? ff >> 1 : d >> 1;
        // weights go out before anything else: they depend on nothing, and come from the farthest
        PkWeights<FWT> w;
        pk_weights<FWT, QT == 1>(w, pk_ptr<pk_cw_t>(rec, 0) + ((long)nt * (down ? ff >> 5 : d >> 5) + kq * KT) * 512, KT);
        const pk_x_t in = pk_ptr<pk_x_t>(rec, 1) + (long)row0 * lda + kq * (ff >> 3), sq0 = pk_ptr<pk_x_t>(rec, 2), hold = pk_ptr<pk_x_t>(rec, 3);
        const pk_x_t to = pk_ptr<pk_x_t>(rec, 4), to_x = pk_ptr<pk_x_t>(rec, 5), to_s = pk_ptr<pk_x_t>(rec, 6);
        const pk_x_t w2p = a.w2part + (((long)nt << rgs) + (u & rgs)) * 768;
        // this thread's place in the tile: row of the group, column
        const int tid = pk_tid(), er = ((tid & 63) >> 4) * 4 + (tid >> 6), n = nt * 16 + (tid & 15), rr_ = min(er, Rl - 1);
        const bool res = goes_on && gi < 6 && kq == 0;
        // The residual operand of a tile (complete long before the tile's GEMM input is) and what else the epilogue needs is requested here and looked at
        // behind the multiplication; only then, if the operand was not there yet, it is waited for.
        u32x2 ov = u32x2{0u, 0u};
        float gain = 0.f;
        f32x2 rot = f32x2{1.f, 0.f};
        const int part = gi > 0 ? 0 : nt >= d >> 3 ? 2 : nt >= d >> 4 ? 1 : 0, cp = nt * 16 - part * d;
        if (res) ov = ld_agent2(pk_buf(hold + (long)row0 * d, Rl * d * 8), (rr_ * d + n) * 8);
        if (goes_on && to_x && kq == 0) gain = pk_ptr<pk_cf_t>(rec, 7)[n];
        if (gi == 0 && part < 2) rot = pk_ptr<const PK_GLOBAL f32x2*>(rec, 7)[(long)(row0 + rr_) * 32 + ((cp & 63) >> 4) * 8 + (tid & 7)];
        float c;
        pk_gemm_tile<FWT>(a, sh, par, w, KT, in, lda, tag, sq0 ? sq0 + (long)row0 * (d >> 4) : sq0, Rl, c, stage);
        const bool on = er < Rl;
        if (goes_on && kq == 0) {
          bool ok = true;
          if (down) {
            unsigned pr[3];
            ok = pk_fetch<3>(pr, 3, on, tag, [&](int i) { return w2p + i * 256 + tid; }, a, stage);
            PK_MARK(4);
#pragma unroll
            for (int k = 0; k < 3; k++) c += __uint_as_float(pr[k]);
          }
          unsigned raw[1] = {ov[0]};
          if (res && !__all(ov[1] == tag)) ok = pk_fetch<1>(raw, 1, true, tag, [&](int) { return hold + (long)(row0 + rr_) * d + n; }, a, stage) && ok;
          const float old = __uint_as_float(raw[0]), v = res ? old + c : c;
          if (ok) {
            pk_put_row(v, on, er, n, d, to + (long)row0 * d, to_x ? to_x + (long)row0 * (d >> 1) : to_x, to_s + (long)row0 * (d >> 4), gain,
                       down ? tag + 1 : tag);
            // rings: a stack's output (no norm behind it); the input of its last layer, which is what the draft heads of the level start from
            const pk_f_t ring = pk_ptr<pk_f_t>(rec, 8);
            if (ring && on) ring[(long)((P0 + row0 + er) & (lev == 0 ? 31 : lev == 1 ? 15 : 7)) * d + n] = down ? v : old;
          } else sh.bad = 1;
        } else if (goes_on) {
          // Only what quarter 0 waits for: the next layer writes the same partial tiles, maybe with more rows, and a store that nobody has waited for
          // could land on top of one of its.
          if (on) pk_stf(w2p + (kq - 1) * 256 + tid, c, tag);
        } else if (gi == 0) {      // to: queries, to_x, to_s: new keys and values; hold, ring: the caches
          const int hh = cp >> 6;
          const pk_x_t dst = part == 0 ? to + (long)row0 * (d >> 1) + hh * 32 : (part == 1 ? to_x : to_s) + ((long)hh * RS + row0) * 32;
          pk_epi_qkv(dst, part == 1 ? (pk_w_t)hold : pk_ptr<pk_w_t>(rec, 8), c, part, cp, tag, on, rot, P0 + row0 + er, lev == 0 ? a.capb[0] : lev == 1 ? a.capb[1] : a.capb[2], er, d);
        } else if (gi == 7) {
          if (on && n < a.D.V) a.logits[(long)(row0 + er) * a.D.V + n] = c;       // plain memory: later launches read them
        } else {
          const int ld2 = gi == 4 ? ff >> 1 : d >> 1;
          pk_put_half(gi == 4 ? gelu_tanh_f(c) : c, on, er, n, to + (long)row0 * ld2, ld2, tag);
        }
        if (pk_bad(sh)) return;
      }
      PK_NEXT(NT << rgs);
    }
    // ---- the next stage
    if (op < PK_W2) op++;
    else if (op == PK_W2) {
      l++;
      op = l < end ? PK_QKV : st == 4 ? PK_LM : st < 2 && of(nr, st + 1) > 0 ? PK_POOL : PK_UP;
    } else if (op == PK_POOL) op = PK_SHORT;
    else if (op == PK_SHORT) { op = PK_QKV; st++; end = l + a.count[st]; }
    else if (op == PK_UP) op = PK_QKV;
    else break;
  }
}

// The instance of a context: two row groups or one, and the width where the compiler knows it (offsets are constants and no fragment is
// conditional); 640 and 896 and hidden widths other than 4 d take the general one.  Steps with the instance / with the general one, us:
//   blocks of 9   d = 128 500 / 549   256 527 / 575   384 559 / 592   512 573 / 619   768 755 / 794   1024 1439 / 1458
//   blocks of 18          567 / 619       604 / 653       656 / 692       695 / 734       934 / 977        1788 / 1812
// (20, at 768 24 and at 1024 40 blocks, memory 2048 and at 1024 4096, window 4500 and 9000).  The narrow widths are where the general one, which multiplies
// eight fragments a wave whatever the width, loses most: with stages of their own code and fragments behind branches it took 522 and 575 us for the passes of
// 18 tokens at 128 and 384, with the loop 535 and 579, the instances 484 and 539.  (Branches in the loop: 1459 -> 1526 at 1024.)
typedef void (*pk_kernel_t)(PkArgs);
inline pk_kernel_t pk_kernel(const PkArgs& a) {
  const int d = a.ff == 4 * a.D.d ? a.D.d : 0;
  const bool two = a.RS == 32;
  switch (d) {
#define FM_PK(FWT) case FWT * 128: return two ? k_verify_persist<2, FWT> : k_verify_persist<1, FWT>
    FM_PK(1); FM_PK(2); FM_PK(3); FM_PK(4); FM_PK(6); FM_PK(8);
#undef FM_PK
  }
  return two ? k_verify_persist<2, 0> : k_verify_persist<1, 0>;
}
