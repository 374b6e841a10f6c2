// Control kernels of one decode step: row bookkeeping for the verify pass, acceptance, commit,
// draft-row set-up, distribution store and the merge that builds the next block.  Integer work
// and a little fp32; every kernel is a single small launch.
#pragma once
#include "fm_device.h"
#include "fm_progress.h"
#include "fm_kernels_decode.h"

struct InvFreq { double v[64]; };  // base^(-i/(hd/2)) for the hd/2 rotary pairs of a head, computed in double on the host

struct Dims {
  int d, H, V, S, Bm, VB, FB, M;
  int hd;                // head width d / H: 64, 96 or 128
  int capc, capv, capf;  // K/V cache slots per level (rings when a window is set)
  int maxtok;            // longest stream (positions 1 .. maxtok)
  int wc, wv, wf;        // attention window per level in its own positions, 0 = unbounded
  int Dc, m, n;          // draft configuration
  int nspv, nspf;        // SP heads at the point / face level
  int nhfc, nhfv;        // HF parameter sets at the coordinate / vertex level
  int nbins, ban, eos, pad;
  int ruleA;             // rule (A) of the supplement: no point-level prediction at a face split node
  int t0, j0;            // rule (B): first coordinate offset (3, or 0 with the rule off) and first vertex offset (1 / 0)
                         // that own an HF parameter set; offsets below them are left to the coordinate level
};

struct StateDev {
  int *P, *main, *fin, *firedv, *firedf, *basec, *basev, *basef;
  int *vlen, *vtok, *y;
  int* hist;          // [S][maxtok + 1], hist[p] = x_p
  int* budget;        // [1]
  int* alive;         // [1] unfinished sequences; doubles as the run flag of the step
  int* level_rows;    // [3] does a level have a row in this verify pass?  Run flags of its launches (k_verify_setup)
  unsigned long long* acc_hist;  // [3][32]: accepted lengths of steps whose block carried coordinate-level drafts only /
                                 // a fresh point-level prediction / a fresh face-level prediction
  unsigned long long* counters;  // [0] steps, [1] tokens, [2] verify rows with a non-finite logit
  int* kind;                     // [S] which of the three the block built by the last draft was
};

__device__ __forceinline__ int eff_block_len(const StateDev& st, const Dims& D, int s, const int* block_len) {
  if (st.fin[s]) return 0;
  int len = block_len ? block_len[s] : 1;
  len = min(len, D.Bm);
  len = min(len, st.budget[0] - st.P[s]);
  return max(len, 0);
}

// Rows of one verify pass, one workgroup per row (coordinate rows, then vertex, then face rows): position, last visible key of
// the cross-attention, rotary table; every entry follows from the committed state alone.  emb != null: coordinate rows also get
// their embedding as fp32 residual stream and as input of the first projection.  Without a block (both pointers null) every sequence
// feeds its main token alone, what k_merge would write for a step without drafts (8 faces of d = 512 token by token 11.08 -> 10.99 ms); qtok: the
// sampled drafts' record, cleared then (none of them may count as drawn for a later block of the caller's).
template <typename T>
__global__ __launch_bounds__(256) void k_verify_setup(StateDev st, Dims D, InvFreq inv, const int* __restrict__ block_tok,
                                                       const int* __restrict__ block_len, int* pos_c, int* pos_v, int* pos_f,
                                                       int* limx_c, int* limx_v, int* limx_f, float2* cs_c, float2* cs_v,
                                                       float2* cs_f, unsigned* epoch, const T* __restrict__ emb, float* __restrict__ h,
                                                       T* __restrict__ xg, const float* __restrict__ gain, float* __restrict__ ssq, int* __restrict__ qtok) {
  if (epoch && blockIdx.x == 0 && threadIdx.x == 0) *epoch += 1;     // pass counter of the single-launch verify kernel
  if (blockIdx.x == 0 && threadIdx.x < 64) {      // at most 64 sequences, a lane each
    const int q = threadIdx.x < D.S ? (int)threadIdx.x : 0, n = (int)threadIdx.x < D.S ? eff_block_len(st, D, q, block_len) : 0, P0 = st.P[q];
    const bool v = n > 0 && (P0 + 2) / 3 * 3 < P0 + n, f = n > 0 && (P0 + 8) / 9 * 9 < P0 + n;
    const int alive = st.alive[0], anyv = __any(v), anyf = __any(f);
    if (threadIdx.x < 3) st.level_rows[threadIdx.x] = threadIdx.x == 0 ? alive : alive && (threadIdx.x == 1 ? anyv : anyf);
  }
  const int Rc = D.S * D.Bm, Rv = D.S * D.VB;
  const int level = (int)blockIdx.x < Rc ? 0 : (int)blockIdx.x < Rc + Rv ? 1 : 2;
  const int idx = blockIdx.x - (level == 0 ? 0 : level == 1 ? Rc : Rc + Rv);
  const int per = level == 0 ? D.Bm : level == 1 ? D.VB : D.FB, step = level == 0 ? 1 : level == 1 ? 3 : 9;
  const int s = idx / per, i = idx % per;
  const int bt = level != 0 ? 0 : block_tok ? block_tok[idx] : st.main[s];
  const int len = eff_block_len(st, D, s, block_len), P = st.P[s];
  const int q = (P + step - 1) / step + i;
  const int p = step * q < P + len ? q : -1;       // a row the block does not reach is inactive
  const int t = p >= 0 && bt >= 0 && bt < D.V ? bt : D.pad;
  if (threadIdx.x == 0) {
    (level == 0 ? pos_c : level == 1 ? pos_v : pos_f)[idx] = p;
    (level == 0 ? limx_c : level == 1 ? limx_v : limx_f)[idx] = p >= 0 ? D.M - 1 : -1;
    if (level == 0) {
      st.vtok[idx] = t;
      if (!block_len) qtok[idx] = -1;
      if (i == 0) {
        st.vlen[s] = len;
        if (!block_len && !st.fin[s]) st.kind[s] = 0;
      }
    }
  }
  const int np = D.hd >> 1;      // rotary pairs per head
  if ((int)threadIdx.x < np) {
    double sn, c;
    sincos((double)max(p, 0) * inv.v[threadIdx.x], &sn, &c);
    (level == 0 ? cs_c : level == 1 ? cs_v : cs_f)[(long)idx * np + threadIdx.x] = make_float2((float)c, (float)sn);
  }
  if (level == 0 && emb) {
    const T* e = emb + (long)t * D.d;
    for (int n = threadIdx.x * 4; n < D.d; n += 1024) {
      f32x4 v = f32x4{0.f, 0.f, 0.f, 0.f};
      if (p >= 0)
#pragma unroll
        for (int k = 0; k < 4; k++) v[k] = Store<T>::ld(e + n + k);
      put_row4<T>(v, idx, n, D.d, h, xg, gain, ssq);
    }
  }
}

// accepted = 1 + number of leading drafts that equal the backbone's greedy prediction; with sampled decoding 1 + number of
// leading drafts that passed the rejection test.  passed: bit i is about draft i + 1 (below len - 1; a wave's ballot).
// (failed: the forward pass gave up and its logits mean nothing; the accepted length is 0)
__device__ __forceinline__ int accepted_length(unsigned long long passed, int len, bool failed) {
  return len > 0 && !failed ? 1 + min(__ffsll(~passed) - 1, len - 1) : 0;
}

// one wave per sequence, a draft per lane (blocks are at most 27 tokens long)
__global__ __launch_bounds__(64) void k_accept(StateDev st, Dims D, int* __restrict__ accepted_out, const int* __restrict__ accflag,
                                               const unsigned* __restrict__ failed) {
  const int s = blockIdx.x, i = threadIdx.x;
  const bool bad = failed && *failed;
  const int len = st.vlen[s], flag = i < D.Bm ? accflag[s * D.Bm + i] : 0;
  const int a = accepted_length(__ballot(i + 1 < len && flag != 0), len, bad);
  if (i == 0 && accepted_out) accepted_out[s] = a;
}

// Greedy choice of every row of a sequence (lowest index among exact ties, over [0, nlim)), into st.y and sy; the block's tokens into stok: one
// workgroup, one wave per row, 16 values per lane in flight.  `nonfinite` counts rows whose admissible logits
// hold an infinity or a NaN: half-precision activations beyond 65504 overflow silently, and this is where it shows.
__device__ __forceinline__ void choose_rows(const StateDev& st, const Dims& D, int s, const float* __restrict__ logits, int nlim, unsigned long long* nonfinite, int* sy, int* stok) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if ((int)threadIdx.x < D.Bm) stok[threadIdx.x] = st.vtok[s * D.Bm + threadIdx.x];
  for (int i = wave; i < D.Bm; i += 16) {
    const float* x = logits + (long)(s * D.Bm + i) * D.V;
    float bv = -INFINITY;
    int bi = 0x7fffffff;
    bool bad = false;
    for (int i0 = lane; i0 < nlim; i0 += 1024) {
      float v[16];
#pragma unroll
      for (int k = 0; k < 16; k++) v[k] = i0 + 64 * k < nlim ? x[i0 + 64 * k] : 0.f;
#pragma unroll
      for (int k = 0; k < 16; k++)
        if (i0 + 64 * k < nlim) {
          bad |= !(fabsf(v[k]) <= 3.0e38f);
          argmax_merge(bv, bi, v[k], i0 + 64 * k);
        }
    }
    wave_argmax(bv, bi);
    bad = __any(bad);
    if (lane == 0) {
      sy[i] = bi;
      st.y[s * D.Bm + i] = bi;
      if (bad) atomicAdd(nonfinite, 1ull);
    }
  }
  __syncthreads();
}

// What the host may look at while the device runs ahead of it: one pinned word per sequence (fm_progress.h), written by the
// commits of fm_generate.
struct Progress { unsigned long long seq[64]; };

struct SeqState { int len, P, fin, kind, budget; };
__device__ __forceinline__ SeqState read_sequence(const StateDev& st, int s) { return SeqState{st.vlen[s], st.P[s], st.fin[s], st.kind[s], st.budget[0]}; }
struct Committed { int pos, fin, moved; };
// One wave commits sequence s; lane i holds token i of the block and the choice behind it (block past its end: anything).
// An accepted length of 0 (a pass that did not complete) leaves the sequence as it is.
__device__ __forceinline__ Committed commit_sequence(const StateDev& st, const Dims& D, int s, int i, const SeqState& q, int acc, int tok, int y, bool bad) {
  const bool moves = !bad && q.len > 0 && acc > 0;
  int a = min(acc, q.len);
  const unsigned long long ends = __ballot(i >= 1 && i < a && tok == D.eos);      // an accepted EOS draft is not fed: it becomes the main token
  if (ends) a = __ffsll(ends) - 1;
  const int mainTok = __shfl(y, max(a - 1, 0), 64);
  const int now = moves ? (mainTok == D.eos || q.P + a >= q.budget ? 1 : 0) : q.fin;
  if (moves) {
    int* h = st.hist + (long)s * (D.maxtok + 1) + q.P;
    if (i < a) h[i] = tok;
    if (i == 0) {
      h[a] = mainTok;
      st.P[s] = q.P + a;
      st.main[s] = mainTok;
      st.fin[s] = now;
      st.vlen[s] = 0;
      atomicAdd(&st.acc_hist[min(max(q.kind, 0), 2) * 32 + min(a, 31)], 1ull);
      atomicAdd(&st.counters[1], (unsigned long long)a);
    }
  }
  return Committed{moves ? q.P + a : q.P, now, moves};
}
// ... and, with a sequence in each lane that is `on`, what concerns all of them.  prog: null for the caller's own commits.
__device__ __forceinline__ void commit_end(const StateDev& st, int i, bool on, const Committed& m, bool bad, unsigned* commits, Progress* prog) {
  const int alive = __popcll(__ballot(on && !m.fin));
  const bool moved = __any(on && m.moved);
  if (i == 0 && !bad) {
    st.alive[0] = alive;
    if (moved) st.counters[0] += 1;
  }
  if (prog) {
    const unsigned n = progress_next(*commits);       // one wave: read by all lanes before lane 0 writes it
    if (i == 0) *commits = n;
    if (on) __hip_atomic_store(&prog->seq[i], progress_word(n, bad ? 0 : m.fin ? 1 : m.pos + 2), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  }
}

// Greedy choice of every row of a sequence and the accepted length, see choose_rows.
__global__ __launch_bounds__(1024) void k_choose_greedy(StateDev st, Dims D, const float* __restrict__ logits, int nlim,
                                                         int* __restrict__ accepted_out, const unsigned* __restrict__ failed,
                                                         unsigned long long* __restrict__ nonfinite) {
  __shared__ int sy[32], stok[32];
  const int s = blockIdx.x, lane = threadIdx.x & 63;
  const int len = st.vlen[s];
  const bool bad_pass = failed && *failed;
  choose_rows(st, D, s, logits, nlim, nonfinite, sy, stok);
  if (threadIdx.x < 64) {      // a draft per lane
    const int a = accepted_length(__ballot(lane + 1 < min(len, 32) && stok[min(lane + 1, 31)] == sy[min(lane, 31)]), len, bad_pass);
    if (lane == 0 && accepted_out) accepted_out[s] = a;
  }
}

// The commit of every sequence.  A wave per sequence, a token of the block per lane: all a sequence needs is read in one trip.  (A thread per
// sequence that walked its block token by token, and such walks at the end of k_choose_greedy and k_merge: steps of d = 512 578 us instead of 574,
// meshes of d = 256 in fp32 10.95 ms instead of 10.84.)
__global__ __launch_bounds__(1024) void k_commit(StateDev st, Dims D, const int* __restrict__ accepted, const unsigned* __restrict__ failed, unsigned* commits,
                                                 Progress* prog) {
  __shared__ int s_pos[64], s_fin[64], s_moved[64];
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), waves = blockDim.x >> 6, i = threadIdx.x & 63;
  const bool bad = failed && *failed;
  for (int s = wave; s < D.S; s += waves) {
    const int acc = accepted[s], tok = i < D.Bm ? st.vtok[s * D.Bm + i] : 0, y = i < D.Bm ? st.y[s * D.Bm + i] : 0;
    const Committed m = commit_sequence(st, D, s, i, read_sequence(st, s), acc, tok, y, bad);
    if (i == 0) { s_pos[s] = m.pos; s_fin[s] = m.fin; s_moved[s] = m.moved; }
  }
  __syncthreads();
  if (wave != 0) return;
  const int q = min(i, D.S - 1);      // a sequence per lane: at most 64
  commit_end(st, i, i < D.S, Committed{s_pos[q], s_fin[q], s_moved[q]}, bad, commits, prog);
}

// One sequence, greedy: choice, acceptance and commit in one launch (fm_generate).  A launch of this size costs 1.7 us a step: 8 faces of
// d = 512 token by token 10.99 -> 10.87 ms, a mesh of ten faces of d = 256 in fp32 10.56 -> 10.51.
__global__ __launch_bounds__(1024) void k_choose_commit(StateDev st, Dims D, const float* __restrict__ logits, int nlim, int* __restrict__ accepted_out,
                                                        const unsigned* __restrict__ failed, unsigned long long* __restrict__ nonfinite, unsigned* commits, Progress* prog) {
  __shared__ int sy[32], stok[32];
  const int i = threadIdx.x & 63;
  const SeqState q = read_sequence(st, 0);
  const bool bad = failed && *failed;
  choose_rows(st, D, 0, logits, nlim, nonfinite, sy, stok);
  if (threadIdx.x >= 64) return;
  const int a = accepted_length(__ballot(i + 1 < min(q.len, 32) && stok[min(i + 1, 31)] == sy[min(i, 31)]), q.len, bad);
  if (i == 0) accepted_out[0] = a;
  const Committed m = commit_sequence(st, D, 0, i, q, a, i < D.Bm ? stok[min(i, 31)] : 0, i < D.Bm ? sy[min(i, 31)] : 0, bad);
  commit_end(st, i, i == 0, m, bad, commits, prog);
}

// End of fm_generate: x_1 .. of every sequence and its length to the caller, counters to pinned host memory.
__global__ __launch_bounds__(256) void k_finish(StateDev st, Dims D, int* __restrict__ out_tok, int* __restrict__ out_len,
                                                unsigned long long* __restrict__ host_counts) {
  const int s = blockIdx.y;
  const int* h = st.hist + (long)s * (D.maxtok + 1) + 1;
  for (int i = blockIdx.x * 256 + threadIdx.x; i < D.maxtok; i += gridDim.x * 256) out_tok[(long)s * D.maxtok + i] = h[i];
  if (blockIdx.x == 0 && threadIdx.x == 0) out_len[s] = st.P[s];
  if (blockIdx.x == 0 && s == 0 && threadIdx.x < 99) host_counts[threadIdx.x] = threadIdx.x < 3 ? st.counters[threadIdx.x] : st.acc_hist[threadIdx.x - 3];
}

// New token budget: sequences that have not ended with EOS become live again if they are below it.
// generation > 0: the start of fm_generate call number `generation` (statistics and the commit counter start over)
__global__ void k_set_budget(StateDev st, Dims D, int budget, unsigned generation, unsigned* commits) {
  if (generation) {
    if (threadIdx.x == 0) *commits = progress_start(generation);
    for (int i = threadIdx.x; i < 96; i += 64) st.acc_hist[i] = 0;
    if (threadIdx.x < 3) st.counters[threadIdx.x] = 0;
  }
  if (threadIdx.x != 0) return;
  st.budget[0] = budget;
  int alive = 0;
  for (int i = 0; i < D.S; i++) {
    if (st.P[i] >= 0 && st.hist[(long)i * (D.maxtok + 1)] == D.nbins)   // sequence has been prefilled
      st.fin[i] = (st.main[i] == D.eos || st.P[i] >= budget) ? 1 : 0;
    alive += st.fin[i] ? 0 : 1;
  }
  st.alive[0] = alive;
}

// A new sequence: its condition memory [M][d] goes into operand order (fragments as k_tile_weight lays out weights, zero rows up to whole key
// blocks) and its state starts over (x_0 = BOS, empty caches, no draft rows).  Workgroup (x, y): rows 16x..+16, a wave per 32 columns; a fragment is one trip, all of them
// are in flight at once.  At d = 1024, 4096 rows 9.5 us for 24 MB, cold; as a
// grid-stride loop with 64-bit divisions and a launch of its own for the state 14 + 4.6 (two sequences of d = 768 with their first block 1195 -> 1186 us).
template <typename T>
__global__ __launch_bounds__(256) void k_admit(const float* __restrict__ mem, T* __restrict__ Xt, int M, int d, StateDev st, Dims D, int s, int bos) {
  if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x < 64) {
    const int i = threadIdx.x;
    const int alive = __popcll(__ballot(i < D.S && (i == s || !st.fin[min(i, D.S - 1)])));      // at most 64 sequences, a lane each
    if (i == 0) {
      st.P[s] = 0; st.main[s] = bos; st.fin[s] = 0;
      st.firedv[s] = -1; st.firedf[s] = -1;
      st.basec[s] = -1000000; st.basev[s] = -1; st.basef[s] = -1;
      st.vlen[s] = 0;
      st.hist[(long)s * (D.maxtok + 1)] = bos;
      st.alive[0] = alive;
    }
  }
  const int KT = d >> 5, kt = blockIdx.y * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  if (kt >= KT) return;
  *reinterpret_cast<typename Op<T>::V8*>(Xt + (((long)blockIdx.x * KT + kt) * 64 + lane) * 8) = tile_part<T>(mem, M, d, blockIdx.x, kt, lane, 0, 1);
}


// ------------------------------------------------------------------------------------------
// Sampled decoding with non-greedy verification: drafts drawn from the averaged draft distributions, the
// rejection test of speculative sampling on the backbone's tempered softmax, residual resampling.
// Uniforms are counter based: (seed, sequence, absolute position of the token decided, purpose).
// ------------------------------------------------------------------------------------------
#define FM_U_DRAFT 0
#define FM_U_ACCEPT 1
#define FM_U_RESAMPLE 2

// Settings that a caller may change between steps.  They live in device memory (k_set_params writes them in stream order), so
// that a step recorded as a graph stays valid when they change.
struct Replay {
  const int* stream;  // [S][stride], stream[p - 1] = x_p
  int stride, n_valid;
  float keep;
  unsigned long long seed;
};
struct StepParams {
  Replay replay;
  float temperature;            // 0 = greedy decoding
  unsigned long long seed;      // of the sampled decoding
  int keep_rows;                // test hook: greedy decoding also leaves the averaged rows in qrow (read by fm_debug_draft)
};
__global__ void k_set_params(StepParams* dst, StepParams v) {
  if (threadIdx.x == 0) *dst = v;
}

struct Sampling {
  const StepParams* p;
  float* qrow;                  // [S][Bm][V] averaged draft distribution behind draft index i (unnormalised over the admissible tokens)
  float* qsum;                  // [S][Bm]    its sum over the admissible tokens
  int* qtok;                    // [S][Bm]    the token drawn from it (-1: none)
  int* accflag;                 // [S][Bm]    row i: draft i + 1 passed the rejection test
};

__device__ __forceinline__ float sample_uniform(unsigned long long seed, int purpose, int seq, int pos);

// inclusive prefix sum over the lanes of a wave
__device__ __forceinline__ float wave_scan(float v) {
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const float u = __shfl_up(v, o, 64);
    if (lane >= o) v += u;
  }
  return v;
}

// Inverse CDF in index order over n weights by one wave: lane t owns the contiguous chunk [t*chunk, (t+1)*chunk); `wf(i)`
// gives weight i.  Returns, in every lane, the smallest i whose cumulative weight exceeds u * total (the last index with weight
// if rounding leaves none).
// KEPT > 0: the weights of a lane are asked for together and stay in registers (up to 64 KEPT weights in all): the second walk ends at the
// pick, and a load in each of its rounds is a trip of its own (k_sample_rows 12.3 -> 11.1 us at 1024 weights).  Sums in index order either way.
template <int KEPT, class F>
__device__ __forceinline__ int wave_inverse_cdf(int n, float u, F wf, float& total) {
  const int lane = threadIdx.x & 63;
  const int chunk = (n + 63) / 64;
  const int i0 = min(lane * chunk, n), i1 = min(i0 + chunk, n);
  const bool kept = chunk <= KEPT;
  float w[KEPT > 0 ? KEPT : 1];
  if (kept) {
#pragma unroll
    for (int k = 0; k < KEPT; k++) w[k] = k < chunk ? wf(min(i0 + k, n - 1)) : 0.f;
  }
  float local = 0.f;
  int last = -1;
  if (kept) {
#pragma unroll
    for (int k = 0; k < KEPT; k++)
      if (i0 + k < i1) {
        local += w[k];
        if (w[k] > 0.f) last = i0 + k;
      }
  } else {
    for (int i = i0; i < i1; i++) {
      const float x = wf(i);
      local += x;
      if (x > 0.f) last = i;
    }
  }
  const float incl = wave_scan(local), excl = incl - local;
  total = __shfl(incl, 63, 64);
  const float thr = u * total;
  int pick = 0x7fffffff;
  if (i0 < i1 && incl > thr) {
    float run = excl;
    if (kept) {
#pragma unroll
      for (int k = 0; k < KEPT; k++)
        if (i0 + k < i1) {
          run += w[k];
          if (run > thr && pick == 0x7fffffff) pick = i0 + k;
        }
    } else {
      for (int i = i0; i < i1; i++) {
        run += wf(i);
        if (run > thr) { pick = i; break; }
      }
    }
    if (pick == 0x7fffffff) pick = last >= 0 ? last : i1 - 1;      // rounding between the chunk's sum and its walk
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    pick = min(pick, __shfl_xor(pick, o, 64));
    last = max(last, __shfl_xor(last, o, 64));
  }
  return pick != 0x7fffffff ? pick : max(last, 0);
}

// ------------------------------------------------------------------------------------------
// Draft stage
// ------------------------------------------------------------------------------------------
struct DraftRows {
  // five row sets: 0 SP coordinate, 1 SP point, 2 SP face, 3 HF vertex, 4 HF coordinate
  const float** src[5];
  int* lim[5];
  int* limx[5];
  float2* cs[5];
  int *alive, *firev, *firef;   // [S]
  int* flags;                   // [0] any alive with P > 0, [1] any face firing
  int rs[5];                    // rows per sequence in the tables of a set: row (sequence s, head k) = s * rs + k.  The
                                // set's own head count, or for the three SP sets the head count of all three together
                                // when their tables are one table (point, face, coordinate heads behind each other)
};

struct DraftBufs {
  const float *tap_c, *tap_v, *tap_f, *ring_yf;   // rings
  const float *spv_out, *spf_out, *hfv_out;        // head outputs feeding the HF blocks
  int spv_rs, spf_rs;                               // rows per sequence in spv_out / spf_out (as DraftRows::rs)
};

__device__ __forceinline__ void set_row(const DraftRows& R, int set, int r, const float* src, int pos, int lim, int M,
                                        const InvFreq& inv, int lane32, int np = 32) {
  if (lane32 == 0) {
    R.src[set][r] = src;
    R.lim[set][r] = lim;
    R.limx[set][r] = lim >= 0 ? M - 1 : -1;
  }
  for (int i = lane32; i < np; i += 32) {        // np = rotary pairs per head
    double sn, c;
    sincos((lim >= 0 ? (double)pos : 0.0) * inv.v[i], &sn, &c);
    R.cs[set][(long)r * np + i] = make_float2((float)c, (float)sn);
  }
}

// 32 threads per row, eight rows per workgroup, workgroups (sequence, row chunk).  The two launch flags (any sequence alive / firing at the
// face level) depend on the committed state only, so every workgroup could derive them; workgroup 0
// does, for all sequences, and writes them.
__global__ __launch_bounds__(256) void k_draft_setup(StateDev st, Dims D, InvFreq inv, DraftRows R, DraftBufs B) {
  const int lane32 = threadIdx.x & 31, grp = threadIdx.x >> 5;  // 8 groups of 32
  const int d = D.d;
  auto predicates = [&](int s, bool& alive, bool& firev, bool& firef, int& spos, int& v, int& f) {
    const int P = st.P[s];
    alive = !st.fin[s] && P > 0;
    spos = P - 1;
    v = alive ? spos / 3 : 0;
    f = alive ? spos / 9 : 0;
    firev = alive && D.m > 0 && ((v % 3) != 0 || !D.ruleA) && st.firedv[s] != v;
    firef = alive && D.n > 0 && st.firedf[s] != f;
  };
  if (blockIdx.x == 0 && blockIdx.y == 0) {
    __shared__ int f_any[2];
    if (threadIdx.x < 2) f_any[threadIdx.x] = 0;
    __syncthreads();
    for (int s = threadIdx.x; s < D.S; s += blockDim.x) {
      bool alive, firev, firef; int spos, v, f;
      predicates(s, alive, firev, firef, spos, v, f);
      if (alive) atomicOr(&f_any[0], 1);
      if (firef) atomicOr(&f_any[1], 1);
    }
    __syncthreads();
    if (threadIdx.x < 2) R.flags[threadIdx.x] = f_any[threadIdx.x];
  }
  {
    const int s = blockIdx.x;
    bool alive, firev, firef; int spos, v, f;
    predicates(s, alive, firev, firef, spos, v, f);
    if (blockIdx.y == 0 && threadIdx.x == 0) { R.alive[s] = alive; R.firev[s] = firev; R.firef[s] = firef; }
    const float* tapc = B.tap_c + ((long)s * 32 + (spos & 31)) * d;
    const float* tapv = B.tap_v + ((long)s * 16 + (v & 15)) * d;
    const float* tapf = B.tap_f + ((long)s * 8 + (f & 7)) * d;
    const float* yf = B.ring_yf + ((long)s * 8 + (f & 7)) * d;
    // row of this thread group: the five sets behind each other
    int q = blockIdx.y * 8 + grp;
    if (q < D.Dc) {                    // set 0: coordinate SP heads k = 1..Dc on the coordinate tap at s
      set_row(R, 0, s * R.rs[0] + q, tapc, spos, alive ? spos : -1, D.M, inv, lane32, D.hd >> 1);
      return;
    }
    q -= D.Dc;
    if (q < D.nspv) {                  // set 1: point SP heads on the vertex tap of v
      set_row(R, 1, s * R.rs[1] + q, tapv, v, firev ? v : -1, D.M, inv, lane32, D.hd >> 1);
      return;
    }
    q -= D.nspv;
    if (q < D.nspf) {                  // set 2: face SP heads on the face tap of f
      set_row(R, 2, s * R.rs[2] + q, tapf, f, firef ? f : -1, D.M, inv, lane32, D.hd >> 1);
      return;
    }
    q -= D.nspf;
    if (q < D.nhfv) {                  // set 3: vertex-level HF, vertex offsets j = j0..n/3-1 from vertex token 3f; input = face feature j/3
      const int j = q + D.j0;
      const float* src = (j < 3) ? yf : B.spf_out + ((long)s * B.spf_rs + (j / 3 - 1)) * d;
      set_row(R, 3, s * D.nhfv + q, src, 3 * f + j, firef ? 3 * f : -1, D.M, inv, lane32, D.hd >> 1);
      return;
    }
    q -= D.nhfv;
    if (q < 2 * D.nhfc) {              // set 4: coordinate-level HF, offsets t = t0..; pipe 0 = point pipeline, pipe 1 = face pipeline
      const int pipe = q / D.nhfc, t = q % D.nhfc + D.t0;
      const int r = s * 2 * D.nhfc + q;
      if (pipe == 0) {
        const bool on = firev && t < D.m;
        // offsets 0..2 (rule (B) off) belong to the current vertex: its own feature; later ones to the SP head outputs
        const float* src = t < 3 ? tapv : B.spv_out + ((long)s * B.spv_rs + min(t / 3 - 1, max(D.nspv - 1, 0))) * d;
        set_row(R, 4, r, src, 3 * v + t, on ? 3 * v : -1, D.M, inv, lane32, D.hd >> 1);
      } else {
        const bool on = firef && t < D.n;
        const float* src = B.hfv_out + ((long)s * max(D.nhfv, 1) + min(max(t / 3 - D.j0, 0), max(D.nhfv - 1, 0))) * d;
        set_row(R, 4, r, src, 9 * f + t, on ? 9 * f : -1, D.M, inv, lane32, D.hd >> 1);
      }
    }
  }
}

// softmax of one LM row of the draft heads into the distribution store of its level
__global__ __launch_bounds__(256) void k_dist_store(const float* __restrict__ logits, Dims D, DraftRows R, float* dist_c,
                                                     float* dist_v, float* dist_f) {
  const int r = blockIdx.x;
  float* dst = nullptr;
  if (r < D.S * D.Dc) {
    const int s = r / D.Dc, k = r % D.Dc;
    if (R.alive[s]) dst = dist_c + ((long)s * D.Dc + k) * D.V;
  } else {
    const int rr = r - D.S * D.Dc;
    const int s = rr / (2 * D.nhfc), q = rr % (2 * D.nhfc);
    const int pipe = q / D.nhfc, t = q % D.nhfc + D.t0;
    if (pipe == 0 && R.firev[s] && t < D.m) dst = dist_v + ((long)s * D.nhfc + (t - D.t0)) * D.V;
    if (pipe == 1 && R.firef[s] && t < D.n) dst = dist_f + ((long)s * D.nhfc + (t - D.t0)) * D.V;
  }
  if (!dst) return;
  const float* x = logits + (long)r * D.V;
  __shared__ float red[4];
  // the first 2048 logits stay in registers between the two passes
  float v[8];
#pragma unroll
  for (int k = 0; k < 8; k++) v[k] = (int)threadIdx.x + 256 * k < D.V ? x[threadIdx.x + 256 * k] : -INFINITY;
  float mx = -INFINITY;
#pragma unroll
  for (int k = 0; k < 8; k++) mx = fmaxf(mx, v[k]);
  for (int i = threadIdx.x + 2048; i < D.V; i += 256) mx = fmaxf(mx, x[i]);
  mx = wave_max(mx);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = mx;
  __syncthreads();
  mx = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
  __syncthreads();
  float sum = 0.f;
#pragma unroll
  for (int k = 0; k < 8; k++) { v[k] = expf(v[k] - mx); sum += v[k]; }
  for (int i = threadIdx.x + 2048; i < D.V; i += 256) sum += expf(x[i] - mx);
  sum = wave_sum(sum);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = sum;
  __syncthreads();
  sum = red[0] + red[1] + red[2] + red[3];
  const float inv = 1.0f / sum;
#pragma unroll
  for (int k = 0; k < 8; k++) if ((int)threadIdx.x + 256 * k < D.V) dst[threadIdx.x + 256 * k] = v[k] * inv;
  for (int i = threadIdx.x + 2048; i < D.V; i += 256) dst[i] = expf(x[i] - mx) * inv;
}

__device__ __forceinline__ float replay_uniform(unsigned long long seed, unsigned long long seq, unsigned long long pos) {
  unsigned long long z = seed * 0x9E3779B97F4A7C15ull + seq * 0xBF58476D1CE4E5B9ull + pos * 0x94D049BB133111EBull +
                         0x2545F4914F6CDD1Dull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  z = z ^ (z >> 31);
  return (float)(z >> 40) * (1.0f / 16777216.0f);
}

__device__ __forceinline__ float sample_uniform(unsigned long long seed, int purpose, int seq, int pos) {
  return replay_uniform(seed * 3ull + (unsigned long long)purpose, (unsigned long long)seq, (unsigned long long)pos);
}

// One workgroup per verify row (sequence s, block index i): the backbone's distribution p = softmax(logits / T) over the
// admissible tokens, the rejection test for the draft at index i + 1 (u q(x) < p(x); a draft that is not the token
// drawn from the stored distribution counts as a proposal with all its mass on it), and the token emitted after this
// row if the accepted prefix ends here: from max(p - q, 0) after a rejection, from p after the last row.
__global__ __launch_bounds__(256) void k_sample_rows(StateDev st, Dims D, const float* __restrict__ logits, Sampling sm) {
  __shared__ float sh[4];
  const int row = blockIdx.x, s = row / D.Bm, i = row % D.Bm;
  const int len = st.vlen[s];
  if (i >= len) return;
  const int nlim = D.ban ? D.nbins : D.V;
  const float* x = logits + (long)row * D.V;
  const unsigned long long seed = sm.p->seed;
  const float invT = fminf(1.0f / sm.p->temperature, 3.0e38f);      // temperature 0 (set after the step was recorded): all mass on the maximum
  // max and sum of exp((x - max) / T)
  float mx = -INFINITY;
  for (int j = threadIdx.x; j < nlim; j += 256) mx = fmaxf(mx, x[j]);
  mx = wave_max(mx);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = mx;
  __syncthreads();
  mx = fmaxf(fmaxf(sh[0], sh[1]), fmaxf(sh[2], sh[3]));
  __syncthreads();
  float sum = 0.f;
  for (int j = threadIdx.x; j < nlim; j += 256) sum += expf((x[j] - mx) * invT);
  // an infinity or a NaN among the logits shows in the sum (inf - inf, or NaN itself)
  sum = wave_sum(sum);
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = sum;
  __syncthreads();
  const float invZp = 1.0f / (sh[0] + sh[1] + sh[2] + sh[3]);
  if (threadIdx.x == 0 && !(fabsf(invZp) <= 3.0e38f && fabsf(mx) <= 3.0e38f)) atomicAdd(st.counters + 2, 1ull);
  __syncthreads();
  auto pf = [&](int j) { return expf((x[j] - mx) * invT) * invZp; };
  const int pos = st.P[s] + i + 1;                       // the token this row decides
  const bool has_draft = i + 1 < len;
  const int xd = has_draft ? st.vtok[s * D.Bm + i + 1] : -1;
  const bool fromq = has_draft && xd == sm.qtok[s * D.Bm + i + 1] && xd >= 0 && xd < nlim;
  const float* q = sm.qrow + ((long)s * D.Bm + i + 1) * D.V;
  const float invZq = fromq ? 1.0f / sm.qsum[s * D.Bm + i + 1] : 0.f;
  bool accepted = false;
  if (has_draft && xd >= 0 && xd < nlim) {
    const float pa = pf(xd), qa = fromq ? q[xd] * invZq : 1.0f;
    accepted = sample_uniform(seed, FM_U_ACCEPT, s, pos) * qa < pa;
  }
  const float u = sample_uniform(seed, FM_U_RESAMPLE, s, pos);
  if (threadIdx.x >= 64) return;      // the draw is one wave's work
  float tot = 0.f;
  int y;
  if (!has_draft) {
    y = wave_inverse_cdf<20>(nlim, u, pf, tot);
  } else {
    auto wf = [&](int j) { return fromq ? fmaxf(pf(j) - q[j] * invZq, 0.f) : (j == xd ? 0.f : pf(j)); };
    y = wave_inverse_cdf<20>(nlim, u, wf, tot);
    // all the mass can vanish only if p and q agree everywhere (or p sits on the draft alone): then p itself
    if (!(tot > 0.f)) y = wave_inverse_cdf<20>(nlim, u, pf, tot);
  }
  if (threadIdx.x == 0) {
    st.y[row] = y;
    sm.accflag[row] = accepted ? 1 : 0;
  }
}

// One workgroup per sequence: update the draft bookkeeping, average the distributions that cover each future position and
// take the greedy (or draw the sampled) token, one wave per draft index; the block ends at the first uncovered position.
// Everything the state holds is read in one trip, the rows of an index in another.
__global__ __launch_bounds__(1024) void k_merge(StateDev st, Dims D, DraftRows R, const float* __restrict__ dist_c,
                                                const float* __restrict__ dist_v, const float* __restrict__ dist_f,
                                                int speculative, int* __restrict__ block_tok,
                                                int* __restrict__ block_len, Sampling sm) {
  __shared__ int stok[32];
  const int s = blockIdx.x, wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const StepParams pr = *sm.p;
  const Replay& rp = pr.replay;
  const int fin = st.fin[s], P = st.P[s], budget = st.budget[0], mainTok = st.main[s];
  const int firev = R.firev[s], firef = R.firef[s], oldv = st.basev[s], oldf = st.basef[s];
  int* tok = block_tok + (long)s * D.Bm;
  const bool sampled = pr.temperature > 0.f;
  if (sampled && (int)threadIdx.x < D.Bm) sm.qtok[s * D.Bm + threadIdx.x] = -1;
  if (fin) {
    if (threadIdx.x == 0) block_len[s] = 0;
    return;
  }
  if (threadIdx.x == 0) tok[0] = mainTok;
  if (P == 0 || !speculative) {
    if (threadIdx.x == 0) { block_len[s] = 1; st.kind[s] = 0; }
    return;
  }
  // synthetic draft source: the known continuation, each token kept with probability `keep`
  const int n_replay = rp.stream ? max(min(D.Bm - 1, min(budget - 1 - P, rp.n_valid - P)), 0) : 0;
  const int t = threadIdx.x;
  const int truth = t >= 1 && t <= n_replay ? rp.stream[(long)s * rp.stride + P + t - 1] : 0;
  const int spos = P - 1;
  const int basec = spos;
  const int basev = firev ? 3 * (spos / 3) : oldv;
  const int basef = firef ? 9 * (spos / 9) : oldf;
  __syncthreads();   // every thread has read the old state
  if (threadIdx.x == 0) {
    st.basec[s] = basec; st.basev[s] = basev; st.basef[s] = basef;
    if (firev) st.firedv[s] = spos / 3;
    if (firef) st.firedf[s] = spos / 9;
    st.kind[s] = firef ? 2 : firev ? 1 : 0;
  }
  const int nlim = D.ban ? D.nbins : D.V;
  for (int idx = 1 + wave; idx < D.Bm; idx += 16) {
    // the averaged distributions behind draft index idx (position spos + 1 + idx), if any level covers it
    const int p = spos + 1 + idx;
    const int kc = p - (basec + 2), tv = p - 1 - basev, tf = p - 1 - basef;
    const float* r0 = kc >= 0 && kc < D.Dc ? dist_c + ((long)s * D.Dc + kc) * D.V : nullptr;
    const float* r1 = basev >= 0 && tv >= D.t0 && tv < D.m ? dist_v + ((long)s * D.nhfc + (tv - D.t0)) * D.V : nullptr;
    const float* r2 = basef >= 0 && tf >= D.t0 && tf < D.n ? dist_f + ((long)s * D.nhfc + (tf - D.t0)) * D.V : nullptr;
    const int cnt = (r0 != nullptr) + (r1 != nullptr) + (r2 != nullptr);
    int bi = -1;
    if (cnt > 0) {
      const float inv = 1.0f / (float)cnt;
      float* qr = sampled || pr.keep_rows ? sm.qrow + ((long)s * D.Bm + idx) * D.V : nullptr;
      float bv = -INFINITY;
      bi = 0x7fffffff;
      for (int i0 = lane; i0 < nlim; i0 += 1024) {
        float a[16], b[16], c[16];
#pragma unroll
        for (int k = 0; k < 16; k++) {
          const int i = min(i0 + 64 * k, nlim - 1);
          a[k] = r0 ? r0[i] : 0.f;
          b[k] = r1 ? r1[i] : 0.f;
          c[k] = r2 ? r2[i] : 0.f;
        }
#pragma unroll
        for (int k = 0; k < 16; k++)
          if (i0 + 64 * k < nlim) {
            float v = a[k];
            if (r1) v += b[k];
            if (r2) v += c[k];
            v *= inv;
            argmax_merge(bv, bi, v, i0 + 64 * k);
            if (qr) qr[i0 + 64 * k] = v;
          }
      }
      if (sampled) {
        // the kept row is the proposal that the verify pass tests against; a wave reads back what its own lanes stored
        // (no weights in registers: with the row's values above they do not fit the 128 that 1024 threads leave, and went to scratch memory, 124
        // bytes a lane, in greedy steps too: 33.1 us a launch for five sequences of 18 tokens and 10.7 greedy, against 25.2 and 9.6)
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
        float total;
        bi = wave_inverse_cdf<0>(nlim, sample_uniform(pr.seed, FM_U_DRAFT, s, p), [&](int i) { return qr[i]; }, total);
        if (lane == 0 && p < budget) { sm.qtok[s * D.Bm + idx] = bi; sm.qsum[s * D.Bm + idx] = total; }
      } else {
        wave_argmax(bv, bi);
      }
    }
    if (lane == 0) stok[idx] = bi;
  }
  __syncthreads();
  // the block ends in front of the first index without a token: a lane per index, in every wave
  int len = __ffsll(~__ballot(lane == 0 || (lane < D.Bm && spos + 1 + lane < budget && stok[min(lane, 31)] >= 0))) - 1;
  if (sampled && t >= len && t < D.Bm) sm.qtok[s * D.Bm + t] = -1;
  if (rp.stream) {
    if (t >= 1 && t <= n_replay) {
      const bool keep = replay_uniform(rp.seed, (unsigned long long)s, (unsigned long long)(P + t)) < rp.keep;
      tok[t] = keep ? truth : (truth + 1) % D.nbins;
    } else if (t > n_replay && t >= 1 && t < len) {
      tok[t] = stok[t];
    }
    len = 1 + n_replay;
  } else if (t >= 1 && t < len) {
    tok[t] = stok[t];
  }
  if (threadIdx.x == 0) block_len[s] = len;
}

// ------------------------------------------------------------------------------------------
// Correct stage (Sec. 3.2): label rows of the point-level features, then the integer correction of a draft block
// ------------------------------------------------------------------------------------------
// One wave per point-level feature: softmax of the three label logits W_label f.  Rows 0 .. S*nspv-1 are the
// point pipeline's SP head outputs (vertex v + k), the rest the face pipeline's vertex-level HF outputs (vertex
// 3f + j); a row is stored only when its pipeline fired for the sequence, so older rows stay usable like the
// token distributions do.
__global__ __launch_bounds__(64) void k_label_rows(Dims D, DraftRows R, const float* __restrict__ spv_out, int spv_rs,
                                                    const float* __restrict__ hfv_out, const float* __restrict__ W,
                                                    float* __restrict__ lab_v, float* __restrict__ lab_f) {
  const int r = blockIdx.x, lane = threadIdx.x;
  const float* src;
  float* dst;
  if (r < D.S * D.nspv) {
    const int s = r / D.nspv, k = r % D.nspv;
    if (!R.firev[s]) return;
    src = spv_out + ((long)s * spv_rs + k) * D.d;      // spv_rs rows per sequence in the SP output buffer
    dst = lab_v + (long)r * 3;
  } else {
    const int rr = r - D.S * D.nspv, s = rr / D.nhfv;
    if (!R.firef[s]) return;
    src = hfv_out + (long)rr * D.d;
    dst = lab_f + (long)rr * 3;
  }
  float z[3] = {0.f, 0.f, 0.f};
  for (int i = lane; i < D.d; i += 64) {
    const float x = src[i];
    z[0] = fmaf(W[i], x, z[0]);
    z[1] = fmaf(W[D.d + i], x, z[1]);
    z[2] = fmaf(W[2 * D.d + i], x, z[2]);
  }
#pragma unroll
  for (int k = 0; k < 3; k++) z[k] = wave_sum(z[k]);
  if (lane == 0) {
    const float mx = fmaxf(z[0], fmaxf(z[1], z[2]));
    const float e0 = expf(z[0] - mx), e1 = expf(z[1] - mx), e2 = expf(z[2] - mx);
    const float inv = 1.0f / (e0 + e1 + e2);
    dst[0] = e0 * inv; dst[1] = e1 * inv; dst[2] = e2 * inv;
  }
}

#define FM_LABEL_HIST 0
#define FM_LABEL_NEW 1
#define FM_LABEL_INTRA 2

// One wave per sequence (a block holds at most 27 tokens, i.e. 9 points): labels of the block's points from the
// stored rows, the historical / intra-batch moves in ascending vertex order, then the z-y-x re-sort of the faces
// that consist of draft tokens only.  Integer work on bin coordinates; the main token is never touched.
// Vertex u owns x_{3u+1..3u+3}; block token i is x_{P+i}.
// What bounds it is trips to memory, one behind the other: everything a block needs is read in two (state, then tokens, labels and the
// first 64 historical vertices, one per lane), the moves work on LDS and registers.  (One thread per sequence that walked the history for
// every point: 71 us a step at 64 vertices.)
__global__ __launch_bounds__(64) void k_correct(StateDev st, Dims D, const float* __restrict__ lab_v, const float* __restrict__ lab_f,
                                                int hist_vertices, int* __restrict__ block_tok, const int* __restrict__ block_len,
                                                int* __restrict__ labels_out) {
  __shared__ int stok[36];          // tokens of the block; a point past its end is never looked at
  __shared__ int slab[9], spt[9];
  const int s = blockIdx.x, lane = threadIdx.x;
  int* tok = block_tok + (long)s * D.Bm;
  int* lout = labels_out ? labels_out + (long)s * D.Bm : nullptr;
  const int fin = st.fin[s], P = st.P[s], basev = st.basev[s], basef = st.basef[s];
  const int len = min(block_len[s], D.Bm);
  if (lout && lane < D.Bm) lout[lane] = -1;
  if (fin || len < 4) return;
  const int u0 = (P + 2) / 3, u1 = (P + len - 4) / 3;
  if (u1 < u0) return;
  const int np = u1 - u0 + 1;                    // <= 9
  const int* known = st.hist + (long)s * (D.maxtok + 1);     // x_0 .. x_P (the pending main token is x_P)
  const int nkv = P / 3, h0 = max(0, nkv - hist_vertices);
  auto vertex = [&](int h, int (&k)[3]) {
    k[0] = known[3 * h + 1]; k[1] = known[3 * h + 2]; k[2] = known[3 * h + 3];
  };
  int hv[3] = {0, 0, 0};
  const bool hon = h0 + lane < nkv;
  if (hon) vertex(h0 + lane, hv);
  if (lane < len) stok[lane] = tok[lane];
  const int off = 3 * u0 + 1 - P;                // block index of the first point's z
  if (lane < np) {
    const int u = u0 + lane;
    float a[3] = {0.f, 0.f, 0.f};
    int cnt = 0;
    const int kv = basev >= 0 ? u - basev / 3 : 0;
    if (basev >= 0 && kv >= 1 && kv <= D.nspv) {
      const float* row = lab_v + ((long)s * D.nspv + kv - 1) * 3;
      a[0] += row[0]; a[1] += row[1]; a[2] += row[2];
      cnt++;
    }
    const int jf = basef >= 0 ? u - basef / 3 : 0;
    if (basef >= 0 && jf >= D.j0 && jf < D.j0 + D.nhfv) {
      const float* row = lab_f + ((long)s * D.nhfv + jf - D.j0) * 3;
      a[0] += row[0]; a[1] += row[1]; a[2] += row[2];
      cnt++;
    }
    int l = FM_LABEL_NEW;
    if (cnt > 0) {
      const float inv = 1.0f / (float)cnt;
      const float m0 = a[0] * inv, m1 = a[1] * inv, m2 = a[2] * inv;
      l = 0;
      float best = m0;
      if (m1 > best) { best = m1; l = 1; }
      if (m2 > best) { best = m2; l = 2; }
    }
    slab[lane] = l;
    if (lout) lout[lane] = l;
  }
  __syncthreads();
  if (lane < np) {
    const int* c = stok + off + 3 * lane;
    spt[lane] = c[0] >= 0 && c[0] < D.nbins && c[1] >= 0 && c[1] < D.nbins && c[2] >= 0 && c[2] < D.nbins;
  }
  __syncthreads();
  // Nearest candidate: the smallest distance, among equals the lowest index; -1 = none.  (A candidate at distance 0 is the point
  // itself: moving there changes nothing.)
  auto nearest = [&](long dd, int idx) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
      const long od = __shfl_xor(dd, o, 64);
      const int oi = __shfl_xor(idx, o, 64);
      if (oi >= 0 && (idx < 0 || od < dd || (od == dd && oi < idx))) { dd = od; idx = oi; }
    }
    return idx;
  };
  auto dist = [](const int* c, const int* k) {
    const long dz = c[0] - k[0], dy = c[1] - k[1], dx = c[2] - k[2];
    return dz * dz + dy * dy + dx * dx;
  };
  for (int i = 0; i < np; i++) {
    if (!spt[i]) continue;
    int* c = stok + off + 3 * i;
    if (slab[i] == FM_LABEL_HIST) {
      long best = 0;
      int bh = -1;
      auto offer = [&](const int* k, int h) {
        if (!(k[0] < D.nbins && k[1] < D.nbins && k[2] < D.nbins)) return;
        const long dd = dist(c, k);
        if (bh < 0 || dd < best) { best = dd; bh = h; }
      };
      if (hon) offer(hv, h0 + lane);
      for (int h = h0 + 64 + lane; h < nkv; h += 64) {
        int k[3];
        vertex(h, k);
        offer(k, h);
      }
      bh = nearest(best, bh);
      if (bh >= 0) {
        int k[3] = {__shfl(hv[0], bh - h0, 64), __shfl(hv[1], bh - h0, 64), __shfl(hv[2], bh - h0, 64)};
        if (bh - h0 >= 64) vertex(bh, k);
        __syncthreads();
        if (lane < 3) c[lane] = k[lane];
      }
    } else if (slab[i] == FM_LABEL_INTRA) {
      long best = 0;
      int bw = -1;
      bool same = false;
      if (lane < np && lane != i && spt[lane]) {
        best = dist(c, stok + off + 3 * lane);
        same = best == 0;
        if (slab[lane] == FM_LABEL_NEW && (u0 + lane) / 3 != (u0 + i) / 3) bw = lane;
      }
      same = __any(same);
      bw = nearest(best, bw);
      __syncthreads();
      if (!same && bw >= 0 && lane < 3) c[lane] = stok[off + 3 * bw + lane];
    }
    __syncthreads();
  }
  // faces whose nine tokens are all drafts of this block: vertices in ascending (z, y, x) order, one lane per face
  const int f = (u0 + 2) / 3 + lane;
  if (f < (u1 + 1) / 3) {
    const int i0 = 3 * f - u0;
    if (spt[i0] && spt[i0 + 1] && spt[i0 + 2]) {
      int* c = stok + off + 3 * i0;
      for (int pass = 0; pass < 2; pass++)
        for (int j = 0; j < 2 - pass; j++) {
          int* a = c + 3 * j;
          int* b = a + 3;
          const bool gt = a[0] != b[0] ? a[0] > b[0] : a[1] != b[1] ? a[1] > b[1] : a[2] > b[2];
          if (gt)
            for (int k = 0; k < 3; k++) { const int t = a[k]; a[k] = b[k]; b[k] = t; }
        }
    }
  }
  __syncthreads();
  if (lane >= off && lane < off + 3 * np) tok[lane] = stok[lane];
}
