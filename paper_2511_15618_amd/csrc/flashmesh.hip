// C-ABI library: context, weight loading, and the enqueue logic of draft / verify / commit.
// See include/flashmesh.h for the contract of every entry point.
#include "../../include/flashmesh.h"

#include <hip/hip_runtime.h>

#include <chrono>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <cstdlib>
#include <functional>
#include <string>
#include <thread>
#include <type_traits>
#include <vector>

#include "fm_device.h"
#include "fm_kernels_step.h"
#include "fm_kernels_mfma.h"
#include "fm_kernels_decode.h"
#include "fm_kernels_persist.h"
#include "fm_kernels_prefill.h"

// Staging area of fm_prefill_condition_static: a file-scope device array instead of memory owned by a context, so that
// the call touches no allocator.  Every GPU the library runs on holds its own copy at its own address; the host-side
// name below is only a handle for hipGetSymbolAddress and is never passed to a kernel or a copy.
#define FM_STATIC_SCRATCH_BYTES (16u << 20)
static __device__ __align__(256) unsigned char scratch[FM_STATIC_SCRATCH_BYTES];

#define RS_C 32  // ring sizes (positions kept per sequence) at the coordinate / vertex / face level
#define RS_V 16
#define RS_F 8

namespace {

struct Layer {
  float *g1, *g2, *g3;
  void *wqkv, *wo, *cq, *ckv, *co, *w1, *w2;  // storage type T, [out, in]
  void *Kc, *Vc;                               // [S][H][cap][64]
  void *Km, *Vm;                               // [S][H][M][64]
  int level;                                   // 0 coordinate, 1 vertex, 2 face
};

struct SpLevel {  // SP heads of one level, head-major contiguous so that one grouped GEMM serves all heads
  int cnt;
  float* g;
  void *wq, *wo, *cq, *co, *lin;
};
struct HfLevel {
  int cnt;
  float* g;
  void *wq, *w1, *w2;
};

struct LoadItem { size_t blob_off, n; void* dst; bool f32; int N, K, rope; };  // N, K > 0: linear weight [N, K], the first `rope` rows of queries / keys

// device address of `scratch` on each GPU, looked up once per device (at the first fm_create on it)
std::mutex g_scratch_mu;
void* g_scratch_addr[64] = {};

}  // namespace

struct fm_ctx {
  fm_config cfg;
  Dims D;
  InvFreq inv;
  hipStream_t stream;
  bool bf16;
  size_t esz;
  int ff, hff, Vpad;
  int Rc, Rv, Rf;  // row slots per level
  std::string err;
  std::vector<void*> allocs;
  std::vector<LoadItem> items;
  size_t blob_elems;
  bool weights_loaded;
  std::vector<bool> prefilled;

  // parameters
  void* emb;
  std::vector<Layer> stacks[5];  // cpre, vpre, face, vpost, cpost
  void *short_cv, *short_vf, *lm;
  float* gf;
  SpLevel sp[3];
  SpLevel sp_all;          // the heads of all three levels as one group list, in memory order point, face, coordinate
  const float** lm_src = nullptr;   // rows of the output head's input: coordinate SP head outputs, then coordinate HF outputs
  HfLevel hfc, hfv;
  float* label_w;     // label head of the correct stage [3][d]
  float *lab_v, *lab_f;   // label distributions of the point pipeline [S][nspv][3] and the face pipeline [S][nhfv][3]
  Sampling smp;           // sampled decoding (temperature 0 = greedy): proposals kept between draft and verify
  int correct_hist = 0;   // historical vertices the correct stage looks at; 0 = stage off (no label rows are computed)

  // state
  StateDev st;
  // rings (fp32)
  float *ring_hc, *ring_hv, *ring_yf, *ring_yv, *tap_c, *tap_v, *tap_f;
  // verify scratch
  int *pos[3], *limx[3];
  float2* cs[3];
  float* h[3];
  void* qT;
  float* logits;
  // one launch per operator: per level the input of the next norm's GEMM (x * gain, tiled) and the row sums of
  // squares; attention output and FFN hidden rows (tiled), queries, attention workspace
  void *xg[3], *attX, *midX;
  float* ssq[3];
  float* attn_ws;
  unsigned* attn_arrived;
  void *dX, *dmidX;   // draft heads: tiled rows of a grouped GEMM, FFN hidden rows
  int sp_tiles = 1, hf_tiles[2] = {1, 1};   // row tiles per parameter set: SP heads; HF sets (vertex, coordinate)
  float* stage;       // staging for weight conversion / prefill GEMM output
  size_t stage_elems;
  unsigned char* static_scratch = nullptr;   // this GPU's copy of the file-scope staging array
  // draft scratch
  DraftRows dr;
  DraftBufs db;
  float *spv_out, *spf_out, *hfv_out, *dh, *dlogits;
  float *dist_c, *dist_v, *dist_f;
  void* dq;
  StepParams params{};     // host copy of the settings below, StepParams on the device
  StepParams* params_dev = nullptr;
  int *gen_tok, *gen_len;  // block buffers used by fm_generate
  int* gen_acc;
  unsigned* commits_dev = nullptr;   // number of the fm_generate call and its commits so far (fm_progress.h)
  unsigned generation = 0;           // fm_generate calls so far, 12 bits
  Progress* prog = nullptr;          // pinned, written by k_commit
  unsigned long long* host_counts = nullptr;   // pinned, written by k_finish
  // Recorded launch sequences.  A decode step is several hundred launches whose arguments never change.  Enqueueing one costs the
  // host 2.6 to 4 us, which bounds the step where the kernels are shorter than that; a graph costs it next to nothing, but
  // 7 us of device time of its own.
  struct GraphKey {
    int what;              // G_*
    int flags;             // launches that depend on a setting (speculative, sampling)
    int hist;              // and on the correct stage: its vertices, 0 = off
    const void* p[4];      // caller's buffers
    bool operator==(const GraphKey& o) const { return what == o.what && flags == o.flags && hist == o.hist && !memcmp(p, o.p, sizeof p); }
  };
  struct Graph {
    GraphKey key;
    hipGraphExec_t exec = nullptr;
    unsigned long used = 0;
  };
  std::vector<Graph> graphs;
  unsigned long graph_clock = 0;
  bool graphs_on = true;
  hipStream_t rec_stream = nullptr;   // recording only, nothing runs on it
  enum { E_BEGIN, E_END, E_P0, E_P1, E_P2, E_P3, E_COUNT };
  hipEvent_t ev[E_COUNT] = {};
  bool sticky_error = false;    // a launch wrapper refused its arguments (message in err); reported by the entry point
  // persistent verify kernel (one sequence, block <= 32, half-precision path)
  bool persist;
  int persist_failures = 0;   // times the single-launch kernel gave up (the context then left that path)
  PkArgs pk;
  PrefillLayer* pf_layers = nullptr;   // per-block table of the tiled prefill GEMM (null: per-block launches)
  int pf_n = 0, pf_grid = 0;           // blocks in the table; workgroups of its launch (one per compute unit, multiple of 8)
  unsigned* pk_epoch;      // device: passes so far
  size_t pk_lds;           // dynamic LDS of the persistent kernel (none at present)
  double weight_bytes;
};

namespace {

int fail(fm_ctx* c, int code, const char* fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  if (c) c->err = buf;
  return code;
}

#define HIPCHK(c, expr)                                                                         \
  do {                                                                                          \
    hipError_t e_ = (expr);                                                                     \
    if (e_ != hipSuccess) return fail(c, FM_EHIP, "%s failed: %s", #expr, hipGetErrorString(e_)); \
  } while (0)

template <typename U> int dalloc(fm_ctx* c, U** p, size_t n, bool zero = true) {
  void* q = nullptr;
  const size_t bytes = (n ? n : 1) * sizeof(U);
  if (hipMalloc(&q, bytes) != hipSuccess) {
    (void)hipGetLastError();
    return fail(c, FM_ENOMEM, "hipMalloc of %zu bytes failed", bytes);
  }
  if (zero && hipMemset(q, 0, bytes) != hipSuccess) return fail(c, FM_EHIP, "hipMemset failed");
  c->allocs.push_back(q);
  *p = (U*)q;
  return FM_OK;
}
int dalloc_t(fm_ctx* c, void** p, size_t n) {  // n elements of the storage type
  uint8_t* q;
  int rc = dalloc(c, &q, n * c->esz);
  *p = q;
  return rc;
}
#define TRY(x) do { int rc_ = (x); if (rc_ != FM_OK) return rc_; } while (0)

enum { G_DRAFT = 1, G_VERIFY, G_STEP };
#define FM_GRAPHS 8      // recorded sequences a context keeps (least recently used goes first)

void drop_graphs(fm_ctx* c) {
  for (auto& g : c->graphs) if (g.exec) (void)hipGraphExecDestroy(g.exec);
  c->graphs.clear();
}

void release(fm_ctx* c) {
  drop_graphs(c);
  if (c->rec_stream) (void)hipStreamDestroy(c->rec_stream);
  for (hipEvent_t e : c->ev) if (e) (void)hipEventDestroy(e);
  for (void* p : c->allocs) (void)hipFree(p);
  if (c->prog) (void)hipHostFree(c->prog);
  if (c->host_counts) (void)hipHostFree(c->host_counts);
  delete c;
}

// Runs `enqueue` (launches on c->stream whose arguments follow from `key` alone) as a graph.  The first call with a key launches
// directly unless `now`; the second records and replays, later ones replay.  A stream that the caller is recording takes
// the launches themselves, and so does a context whose recording failed once.
int run_graphed(fm_ctx* c, const fm_ctx::GraphKey& key, bool now, const std::function<int()>& enqueue) {
  if (!c->graphs_on) return enqueue();
  if (c->stream) {
    hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing(c->stream, &cs) != hipSuccess) (void)hipGetLastError();
    if (cs != hipStreamCaptureStatusNone) return enqueue();
  }
  fm_ctx::Graph* g = nullptr;
  for (auto& x : c->graphs) if (x.key == key) g = &x;
  const bool known = g != nullptr;
  if (!g) {
    if (c->graphs.size() >= FM_GRAPHS) {
      size_t old = 0;
      for (size_t i = 1; i < c->graphs.size(); i++) if (c->graphs[i].used < c->graphs[old].used) old = i;
      // the stream may still be working on the launch of the one that goes
      if (c->graphs[old].exec) { HIPCHK(c, hipStreamSynchronize(c->stream)); (void)hipGraphExecDestroy(c->graphs[old].exec); }
      c->graphs[old] = fm_ctx::Graph{};
      g = &c->graphs[old];
    } else {
      c->graphs.emplace_back();
      g = &c->graphs.back();
    }
    g->key = key;
  }
  g->used = ++c->graph_clock;
  if (!g->exec) {
    if (!known && !now) return enqueue();
    hipStream_t user = c->stream;
    hipGraph_t graph = nullptr;
    if (!c->rec_stream && hipStreamCreateWithFlags(&c->rec_stream, hipStreamNonBlocking) != hipSuccess) c->rec_stream = nullptr;
    hipError_t e = c->rec_stream ? hipStreamBeginCapture(c->rec_stream, hipStreamCaptureModeThreadLocal) : hipErrorUnknown;
    int rc = FM_OK;
    if (e == hipSuccess) {
      c->stream = c->rec_stream;
      rc = enqueue();
      c->stream = user;
      e = hipStreamEndCapture(c->rec_stream, &graph);
      if (rc == FM_OK && e == hipSuccess) e = hipGraphInstantiate(&g->exec, graph, nullptr, nullptr, 0);
      if (graph) (void)hipGraphDestroy(graph);
    }
    if (rc != FM_OK) { g->exec = nullptr; return rc; }
    if (e != hipSuccess) {
      (void)hipGetLastError();
      g->exec = nullptr;
      c->graphs_on = false;
      return enqueue();
    }
  }
  HIPCHK(c, hipGraphLaunch(g->exec, c->stream));
  return FM_OK;
}

int level_cap(const fm_ctx* c, int level) { return level == 0 ? c->D.capc : level == 1 ? c->D.capv : c->D.capf; }
int level_window(const fm_ctx* c, int level) { return level == 0 ? c->D.wc : level == 1 ? c->D.wv : c->D.wf; }
const int kStackLevel[5] = {0, 1, 2, 1, 0};

// elements of one (sequence) slice of a K or V cache with `cap` key positions
size_t cache_seq_elems(const fm_ctx* c, int cap) {
  return (size_t)c->D.H * ((cap + 31) / 32) * 32 * c->D.hd;
}

// Word that the single-launch verify kernel raises when one of its bounded waits gave up (null on the per-operator
// path): the acceptance and commit kernels then report 0 accepted tokens and change nothing.
const unsigned* pass_failed(const fm_ctx* c) { return c->persist ? c->pk.abort_word : nullptr; }

int commit_any(fm_ctx* c, const int32_t* accepted, bool report) {
  hipLaunchKernelGGL(k_commit, dim3(1), dim3(64 * std::min(c->D.S, 16)), 0, c->stream, c->st, c->D, accepted, pass_failed(c), c->commits_dev, report ? c->prog : nullptr);
  HIPCHK(c, hipGetLastError());
  return FM_OK;
}

// per verify row: the backbone's greedy token (or, with sampled decoding, the rejection test and the resampled token),
// then the accepted length per sequence; commit (in fm_generate): the commit behind them
int choose_and_accept(fm_ctx* c, const float* logits, int32_t* accepted, bool commit) {
  const Dims& D = c->D;
  if (c->params.temperature > 0.f) {
    hipLaunchKernelGGL(k_sample_rows, dim3(c->Rc), dim3(256), 0, c->stream, c->st, D, logits, c->smp);
    hipLaunchKernelGGL(k_accept, dim3(D.S), dim3(64), 0, c->stream, c->st, D, accepted, (const int*)c->smp.accflag, pass_failed(c));
  } else if (commit && D.S == 1) {      // (more sequences have more rows than the waves of one workgroup)
    hipLaunchKernelGGL(k_choose_commit, dim3(1), dim3(1024), 0, c->stream, c->st, D, logits, D.ban ? D.nbins : D.V, accepted, pass_failed(c),
                       c->st.counters + 2, c->commits_dev, c->prog);
    commit = false;
  } else {
    hipLaunchKernelGGL(k_choose_greedy, dim3(D.S), dim3(1024), 0, c->stream, c->st, D, logits, D.ban ? D.nbins : D.V, accepted, pass_failed(c),
                       c->st.counters + 2);
  }
  HIPCHK(c, hipGetLastError());
  return commit ? commit_any(c, accepted, true) : FM_OK;
}

template <typename T>
void verify_setup(fm_ctx* c, const int32_t* block_tok, const int32_t* block_len, bool embed) {
  const Dims& D = c->D;
  hipLaunchKernelGGL((k_verify_setup<T>), dim3(c->Rc + c->Rv + c->Rf), dim3(256), 0, c->stream, c->st, D, c->inv, block_tok, block_len,
                     c->pos[0], c->pos[1], c->pos[2], c->limx[0], c->limx[1], c->limx[2], c->cs[0], c->cs[1], c->cs[2], c->persist ? c->pk_epoch : nullptr,
                     embed ? (const T*)c->emb : nullptr, c->h[0], (T*)c->xg[0], c->stacks[0][0].g1, c->ssq[0], c->smp.qtok);
}

// ------------------------------------------------------------------------------------------
// One launch per operator (fm_kernels_decode.h), in both storage types
// ------------------------------------------------------------------------------------------
int level_rows(const fm_ctx* c, int level) { return level == 0 ? c->Rc : level == 1 ? c->Rv : c->Rf; }
int level_rps(const fm_ctx* c, int level) { return level == 0 ? c->D.Bm : level == 1 ? c->D.VB : c->D.FB; }

void refuse(fm_ctx* c, const char* what) { fail(c, FM_EINVAL, "%s: unsupported row set", what); c->sticky_error = true; }

// one transformer block on the row set of `level` (Sec. 3.1: self-attention, cross-attention to c, FFN).  next_gain: gain of
// the norm behind the block (null: none reads its output); next_qkv: first weights of the block behind it (may be null).  tap / ring: rings that receive the block's input / output rows.
template <typename T>
void run_block(fm_ctx* c, const Layer& L, int level, const float* next_gain, float* tap, float* ring, int rs, const void* next_qkv) {
  const Dims& D = c->D;
  const int d = D.d, rows = level_rows(c, level), RPS = level_rps(c, level), cap = level_cap(c, level);
  const int* flag = c->st.level_rows + level;
  DecGemm b{};                       // what all GEMMs of the block share
  b.M = rows; b.run_flag = flag; b.eps = c->cfg.rms_eps; b.RPS = RPS; b.H = D.H; b.hd = D.hd;
  auto normed = [&](const void* W, int N) {
    DecGemm a = b;
    a.A = c->xg[level]; a.W = W; a.N = N; a.KT = d / 32; a.ssq = c->ssq[level]; a.inv_k = 1.0f / d;
    return a;
  };
  auto residual = [&](const void* X, const void* W, int K, const float* gain) {
    DecGemm a = b;
    a.A = X; a.W = W; a.N = d; a.KT = K / 32;
    a.Y = c->h[level]; a.ldy = d; a.R = c->h[level]; a.ldr = d;
    a.gain = gain; a.X = gain ? c->xg[level] : nullptr; a.ssq_out = gain ? c->ssq[level] : nullptr;
    return a;
  };
  // Weights that the attention launches read ahead (k_dec_attn): the two projections behind each always; behind the cross-attention all
  // up to the next attention where they and the memory's keys and values stay under 48 MB.  Beyond that the launch is bound by
  // its own stream or L2 (32 MB) does not keep what it read: d = 768 x 3: 1286 -> 1223 us a step with all, 1259 with the projections;
  // d = 1024, one sequence: 2286 -> 2132, 2222; eight sequences (134 MB of keys and values): 3220 -> 3327, 3214; d = 1536 x 4: 4173 -> 4370, 4122.
  const double cross_bytes = sizeof(T) * (2.0 * D.S * D.M * d + 4.0 * d * d + 2.0 * d * c->ff);
  auto attn = [&](const int* limit, void* K, void* V, int kcap, int window, bool cross) {
    AttnArgs t{};
    int n = 0;
    auto ahead = [&](const void* W, int N, int Kw) { if (W) t.next[n++] = WeightRange{W, Kw * 16 * (int)sizeof(T), N / 16}; };
    if (cross) {
      ahead(L.co, d, d);
      if (cross_bytes <= 48e6) { ahead(L.w1, c->ff, d); ahead(L.w2, d, c->ff); ahead(next_qkv, 3 * d, d); }
    } else {
      ahead(L.wo, d, d);
      ahead(L.cq, d, d);
    }
    t.S = D.S; t.H = D.H; t.ws = c->attn_ws; t.arrived = c->attn_arrived; t.run_flag = flag;
    t.set[0] = AttnSet{c->qT, limit, RPS, 0, RPS, K, V, (long)cache_seq_elems(c, kcap), (kcap + 31) / 32, window, 1,
                       RowMap{1, RPS, 0, 0}, c->attX};
    if (!dec_attention<T>(t, 1, D.hd, c->stream)) refuse(c, "attention");
  };
  {
    DecGemm a = normed(L.wqkv, 3 * d);
    a.Y = c->qT; a.ldy = d; a.cs = c->cs[level]; a.pos = c->pos[level];
    a.Kc = L.Kc; a.Vc = L.Vc; a.seq_stride = (long)cache_seq_elems(c, cap); a.capb = (cap + 31) / 32;
    dec_gemm<T, DE_QKV, true>(a, 1, c->stream);
  }
  attn(c->pos[level], L.Kc, L.Vc, cap, level_window(c, level), false);
  {
    DecGemm a = residual(c->attX, L.wo, d, L.g2);
    if (tap) { a.tap = tap; a.pos = c->pos[level]; a.rs = rs; }
    dec_gemm<T, DE_RES, false>(a, 1, c->stream);
  }
  {
    DecGemm a = normed(L.cq, d);
    a.Y = c->qT; a.ldy = d;
    dec_gemm<T, DE_ROW, true>(a, 1, c->stream);
  }
  attn(c->limx[level], L.Km, L.Vm, D.M, 0, true);
  dec_gemm<T, DE_RES, false>(residual(c->attX, L.co, d, L.g3), 1, c->stream);
  {
    DecGemm a = normed(L.w1, c->ff);
    a.X = c->midX;
    dec_gemm<T, DE_GELU, true>(a, 1, c->stream);
  }
  {
    DecGemm a = residual(c->midX, L.w2, c->ff, next_gain);
    if (ring) { a.ring = ring; a.pos = c->pos[level]; a.rs = rs; }
    dec_gemm<T, DE_RES, false>(a, 1, c->stream);
  }
}

// The backbone forward of a pass whose rows k_verify_setup has prepared (embedded rows in h[0], xg[0], ssq[0]).
// The launches of a level without a row in the pass (no sequence begins a vertex or a face: short blocks, one-token decoding) end at once; the finer
// level then takes the coarse outputs of earlier passes from the ring, as its rows always do where their coarse row is an earlier one.
// (A mesh of ten faces in blocks of four tokens, fp32, d = 256: 11.5 -> 11.1 ms; eight faces token by token, d = 512, two and five
// sequences: 43.5 -> 39.5 and 47.9 -> 42.3.  An empty launch is still most of a launch.)
template <typename T>
void forward(fm_ctx* c, float* logits) {
  const Dims& D = c->D;
  const int d = D.d;
  float* tap[5] = {nullptr, nullptr, c->tap_f, c->tap_v, c->tap_c};
  float* ring[5] = {c->ring_hc, c->ring_hv, c->ring_yf, c->ring_yv, nullptr};
  const int rsz[3] = {RS_C, RS_V, RS_F};
  for (int st = 0; st < 5; st++) {
    const int level = kStackLevel[st];
    const size_t n = c->stacks[st].size();
    for (size_t i = 0; i < n; i++) {
      const bool last = i + 1 == n;
      const float* gain = !last ? c->stacks[st][i + 1].g1 : st == 4 ? c->gf : nullptr;
      run_block<T>(c, c->stacks[st][i], level, gain, last ? tap[st] : nullptr, last ? ring[st] : nullptr, rsz[level], !last ? c->stacks[st][i + 1].wqkv : nullptr);
    }
    if (st < 2) {          // shorten onto the next coarser level
      const int cl = st + 1;
      hipLaunchKernelGGL((k_dec_pool3<T>), dim3(level_rows(c, cl)), dim3(256), 0, c->stream, ring[st], rsz[level], c->pos[cl], level_rps(c, cl), (T*)c->attX, d,
                         c->st.level_rows + cl);
      DecGemm a{};
      a.A = c->attX; a.W = st == 0 ? c->short_cv : c->short_vf; a.M = level_rows(c, cl); a.N = d; a.KT = d / 32; a.run_flag = c->st.level_rows + cl;
      a.Y = c->h[cl]; a.ldy = d; a.X = c->xg[cl]; a.gain = c->stacks[st + 1][0].g1; a.ssq_out = c->ssq[cl];
      dec_gemm<T, DE_RES, false>(a, 1, c->stream);
    } else if (st < 4) {   // upsample onto the next finer level (repeat + skip)
      const int fl = level - 1;
      hipLaunchKernelGGL((k_dec_upsample<T>), dim3(level_rows(c, fl)), dim3(256), 0, c->stream, c->h[fl], c->pos[fl], level_rps(c, fl), ring[st], rsz[level], d,
                         (T*)c->xg[fl], c->stacks[st + 1][0].g1, c->ssq[fl], c->st.level_rows + fl);
    }
  }
  DecGemm a{};
  a.A = c->xg[0]; a.W = c->lm; a.M = c->Rc; a.N = D.V; a.KT = d / 32; a.ssq = c->ssq[0]; a.inv_k = 1.0f / d; a.eps = c->cfg.rms_eps;
  a.run_flag = c->st.alive; a.Y = logits; a.ldy = D.V;
  dec_gemm<T, DE_F32, true>(a, 1, c->stream);
}

template <typename T>
int verify_impl(fm_ctx* c, const int32_t* block_tok, const int32_t* block_len, float* logits_out, int32_t* accepted, bool commit) {
  float* lg = logits_out ? logits_out : c->logits;
  verify_setup<T>(c, block_tok, block_len, !c->persist);
  if (c->persist) {
    // the whole backbone forward in one launch (see fm_kernels_persist.h)
    c->pk.logits = (pk_f_t)lg;
    hipLaunchKernelGGL(pk_kernel(c->pk), dim3(PK_NWG), dim3(256), c->pk_lds, c->stream, c->pk);
  } else {
    forward<T>(c, lg);
  }
  HIPCHK(c, hipGetLastError());
  return choose_and_accept(c, lg, accepted, commit);
}

// Query projection of draft rows behind their norm: grouped GEMM over `G` sets of `M` rows each with the rotation applied, row (set g, m) -> m * G + g
// in the tables and in the output
template <typename T>
void draft_query(fm_ctx* c, const float* const* src, const float* gain, const void* W, int M, int G, const RowMap& rm, int per_seq, const float2* cs, const int* flag) {
  const int d = c->D.d;
  DecGemm a{};
  a.W = W; a.gsw = (long)d * d; a.M = M; a.N = d; a.KT = d / 32; a.run_flag = flag; a.eps = c->cfg.rms_eps;
  a.Y = c->dq; a.ldy = (long)G * d; a.gsy = d; a.cs = cs; a.ldc = G; a.hd = c->D.hd; a.H = c->D.H;
  a.src = src; a.sgain = gain;
  if (dec_gemm_rows<T, DE_ROPE>(a, G, c->stream)) return;
  hipLaunchKernelGGL((k_dec_rmsnorm<T>), dim3(M * G), dim3(256), 0, c->stream, src, gain, G, (T*)c->dX, rm, per_seq, d, c->cfg.rms_eps, flag);
  a.A = c->dX; a.gsa = (long)rm.tiles * 16 * d;
  dec_gemm<T, DE_ROPE, DN_NONE>(a, G, c->stream);
}

// The SP chains (Eq. 1) of all three levels as one chain of grouped launches: the row set is, per sequence, the point-,
// face- and coordinate-level rows behind each other, every GEMM is grouped over all heads (S rows per head), and the
// two attention launches take one cache per level.  Rows of a level that does not fire in this step carry limit -1 (no
// keys) and produce values nobody reads.
template <typename T>
void run_sp(fm_ctx* c, const int* flag) {
  const Dims& D = c->D;
  const SpLevel& A = c->sp_all;
  const int d = D.d, G = A.cnt, S = D.S;
  if (G == 0) return;
  const RowMap rm{G, 1, 0, c->sp_tiles};
  const int nrow[3] = {D.nspv, D.nspf, D.Dc}, lev[3] = {1, 2, 0};
  const Layer* last[3] = {&c->stacks[3].back(), &c->stacks[2].back(), &c->stacks[4].back()};
  auto attn = [&](const int* limit, bool cross) {
    AttnArgs t{};
    t.S = S; t.H = D.H; t.ws = c->attn_ws; t.arrived = c->attn_arrived; t.run_flag = flag;
    int n = 0, q0 = 0;
    for (int z = 0; z < 3; z++) {
      const int cap = cross ? D.M : level_cap(c, lev[z]);
      if (nrow[z] > 0)
        t.set[n++] = AttnSet{c->dq, limit, nrow[z], q0, G, cross ? last[z]->Km : last[z]->Kc, cross ? last[z]->Vm : last[z]->Vc,
                             (long)cache_seq_elems(c, cap), (cap + 31) / 32, cross ? 0 : level_window(c, lev[z]), 1, rm, c->dX};
      q0 += nrow[z];
    }
    if (!dec_attention<T>(t, n, D.hd, c->stream)) refuse(c, "SP attention");
  };
  DecGemm g{};
  g.A = c->dX; g.gsa = (long)c->sp_tiles * 16 * d; g.gsw = (long)d * d; g.M = S; g.N = d; g.KT = d / 32; g.run_flag = flag;
  draft_query<T>(c, c->dr.src[1], A.g, A.wq, S, G, rm, G, c->dr.cs[1], flag);
  attn(c->dr.lim[1], false);
  // output projection of the self-attention, then straight (no norm, Eq. 1) the cross-attention query
  DecGemm a = g;
  a.W = A.wo; a.X = c->dmidX; a.gsx = g.gsa;
  dec_gemm<T, DE_TILE, false>(a, G, c->stream);
  a = g;
  a.A = c->dmidX; a.W = A.cq; a.Y = c->dq; a.ldy = (long)G * d; a.gsy = d;
  dec_gemm<T, DE_ROW, false>(a, G, c->stream);
  attn(c->dr.limx[1], true);
  a = g;
  a.W = A.co; a.X = c->dmidX; a.gsx = g.gsa;
  dec_gemm<T, DE_TILE, false>(a, G, c->stream);
  // outputs: per sequence the point, face and coordinate rows behind each other (spv_out, spf_out and the rows the output
  // head's pointer table names)
  a = g;
  a.A = c->dmidX; a.W = A.lin; a.Y = c->spv_out; a.ldy = (long)G * d; a.gsy = d; a.Rt = c->dr.src[1]; a.ldc = G;
  dec_gemm<T, DE_F32, false>(a, G, c->stream);
}

// HF block chain (Eq. 3-6): row sets 3 (vertex level) and 4 (coordinate level, mult = 2: the point and the face pipeline
// share the parameter sets)
template <typename T>
void run_hf(fm_ctx* c, int set, const HfLevel& hf, int mult, const Layer& last, int level, float* out, const int* flag) {
  const Dims& D = c->D;
  const int d = D.d, G = hf.cnt, per_seq = G * mult, Mg = D.S * mult, tiles = c->hf_tiles[set - 3];
  if (G == 0) return;
  const RowMap rm{G, mult, 0, tiles};
  draft_query<T>(c, c->dr.src[set], hf.g, hf.wq, Mg, G, rm, per_seq, c->dr.cs[set], flag);
  AttnArgs t{};
  t.S = D.S; t.H = D.H; t.ws = c->attn_ws; t.arrived = c->attn_arrived; t.run_flag = flag;
  const int cap = level_cap(c, level);
  int n = 0;
  for (int q0 = 0; q0 < per_seq; q0 += 32)      // at most 54 rows per sequence: one or two sets
    t.set[n++] = AttnSet{c->dq, c->dr.lim[set], std::min(32, per_seq - q0), q0, per_seq, last.Kc, last.Vc,
                         (long)cache_seq_elems(c, cap), (cap + 31) / 32, level_window(c, level), 1, rm, c->dX};
  if (!dec_attention<T>(t, n, D.hd, c->stream)) refuse(c, "HF attention");
  DecGemm a{};
  a.A = c->dX; a.gsa = (long)tiles * 16 * d; a.W = hf.w1; a.gsw = (long)d * c->hff; a.M = Mg; a.N = c->hff; a.KT = d / 32; a.run_flag = flag;
  a.X = c->dmidX; a.gsx = (long)tiles * 16 * c->hff;
  dec_gemm<T, DE_GELU, false>(a, G, c->stream);
  a.A = c->dmidX; a.gsa = a.gsx; a.W = hf.w2; a.N = d; a.KT = c->hff / 32; a.X = nullptr;
  a.Y = out; a.ldy = (long)G * d; a.gsy = d; a.Rt = c->dr.src[set]; a.ldc = G;
  dec_gemm<T, DE_F32, false>(a, G, c->stream);
}

// Output head on the draft rows (coordinate SP heads, then the coordinate HF rows)
template <typename T>
void draft_logits(fm_ctx* c, int n, const int* flag) {
  const Dims& D = c->D;
  DecGemm a{};
  a.W = c->lm; a.M = n; a.N = D.V; a.KT = D.d / 32; a.run_flag = flag; a.Y = c->dlogits; a.ldy = D.V;
  a.src = c->lm_src; a.sgain = c->gf; a.ldc = 1; a.eps = c->cfg.rms_eps;
  if (dec_gemm_rows<T, DE_F32>(a, 1, c->stream)) return;
  hipLaunchKernelGGL((k_dec_rmsnorm<T>), dim3(n), dim3(256), 0, c->stream, c->lm_src, c->gf, 0, (T*)c->dX, RowMap{1, 0, 0, 0}, n, D.d, c->cfg.rms_eps, flag);
  a.A = c->dX;
  dec_gemm<T, DE_F32, DN_NONE>(a, 1, c->stream);
}

template <typename T>
int draft_impl(fm_ctx* c, int32_t* block_tok, int32_t* block_len, int speculative) {
  const Dims& D = c->D;
  const int d = D.d;
  if (speculative) {
    hipLaunchKernelGGL(k_draft_setup, dim3(D.S, (D.Dc + D.nspv + D.nspf + D.nhfv + 2 * D.nhfc + 7) / 8 + (D.Dc + D.nspv + D.nspf + D.nhfv + 2 * D.nhfc == 0)), dim3(256), 0, c->stream, c->st, D, c->inv, c->dr, c->db);
    const int *f_alive = c->dr.flags, *f_f = c->dr.flags + 1;
    const Layer& lastc = c->stacks[4].back();
    const Layer& lastv = c->stacks[3].back();
    const int nLM = D.S * (D.Dc + 2 * D.nhfc);
    run_sp<T>(c, f_alive);
    run_hf<T>(c, 3, c->hfv, 1, lastv, 1, c->hfv_out, f_f);
    if (c->correct_hist > 0 && D.nspv + D.nhfv > 0)     // label rows of the point-level features (Sec. 3.2)
      hipLaunchKernelGGL(k_label_rows, dim3(D.S * (D.nspv + D.nhfv)), dim3(64), 0, c->stream, D, c->dr, c->spv_out, c->db.spv_rs, c->hfv_out,
                         c->label_w, c->lab_v, c->lab_f);
    float* hfc_out = c->dh + (long)D.S * D.Dc * d;
    run_hf<T>(c, 4, c->hfc, 2, lastc, 0, hfc_out, f_alive);
    if (nLM > 0) {
      draft_logits<T>(c, nLM, f_alive);
      hipLaunchKernelGGL(k_dist_store, dim3(nLM), dim3(256), 0, c->stream, c->dlogits, D, c->dr, c->dist_c, c->dist_v,
                         c->dist_f);
    }
  }
  hipLaunchKernelGGL(k_merge, dim3(D.S), dim3(1024), 0, c->stream, c->st, D, c->dr, c->dist_c, c->dist_v, c->dist_f,
                     speculative, block_tok, block_len, c->smp);
  HIPCHK(c, hipGetLastError());
  return FM_OK;
}

int draft_any(fm_ctx* c, int32_t* block_tok, int32_t* block_len, int speculative) {
  return c->bf16 ? draft_impl<f16_t>(c, block_tok, block_len, speculative) : draft_impl<float>(c, block_tok, block_len, speculative);
}
int verify_any(fm_ctx* c, const int32_t* block_tok, const int32_t* block_len, float* logits, int32_t* accepted, bool commit = false) {
  return c->bf16 ? verify_impl<f16_t>(c, block_tok, block_len, logits, accepted, commit) : verify_impl<float>(c, block_tok, block_len, logits, accepted, commit);
}
// settings that decide which launches a step consists of
int step_flags(const fm_ctx* c, int speculative) {
  return (speculative ? 1 : 0) | (c->params.temperature > 0.f ? 2 : 0);
}
int put_params(fm_ctx* c) {
  hipLaunchKernelGGL(k_set_params, dim3(1), dim3(64), 0, c->stream, c->params_dev, c->params);
  HIPCHK(c, hipGetLastError());
  return FM_OK;
}

// staging bytes a prefill call needs: the memory in operand order (whole 32-row blocks) and, where the tiled GEMM does not run
// (fp32, models narrower than it takes), the fp32 K/V rows of one block behind it.  There the two are taken for unpadded
// rows: an area that the padding does not fit takes the keys and the values of a block one after the other (prefill_impl).
size_t prefill_stage_bytes(const fm_ctx* c) {
  const size_t M = c->D.M, d = c->D.d, M32 = (M + 31) / 32 * 32;
  return c->pf_layers ? M32 * d * c->esz : M * d * (c->esz + 2 * sizeof(float));
}

template <typename T>
int prefill_impl(fm_ctx* c, int seq, const float* mem_dev, void* stage_area, size_t stage_bytes) {
  const Dims& D = c->D;
  const int d = D.d, M32 = (D.M + 31) / 32 * 32;
  const size_t tiled = (size_t)M32 * d * sizeof(T), rows = (size_t)D.M * d * sizeof(float);      // memory in operand order; keys or values of one block
  const int parts = tiled + 2 * rows <= stage_bytes ? 1 : 2;       // keys and values of a block together, or in turn
  if (tiled + (c->pf_layers ? 0 : 2 / parts * rows) > stage_bytes) return fail(c, FM_EINVAL, "condition memory of %d x %d does not fit its staging area", D.M, d);
  // memory -> MFMA fragment order; the sequence starts over
  T* Xt = (T*)stage_area;
  hipLaunchKernelGGL((k_admit<T>), dim3(M32 / 16, (d / 32 + 3) / 4), dim3(256), 0, c->stream, mem_dev, Xt, D.M, d, c->st, D, seq, D.nbins);
  const long seq_off = (long)((size_t)seq * cache_seq_elems(c, D.M));
  if (c->pf_layers) {
    // keys and values of one sequence past the last-level cache: as non-temporal stores they leave the memory tiles in L2.
    // Eight sequences of d = 1024 with their first block (671 MB each) 7873 -> 7781 us, two of d = 1536 (302 MB) 2250 -> 2225; two of d = 256 (6 MB) 628 -> 635,
    // where that block then finds nothing in the caches.
    const bool past = 2.0 * c->pf_n * M32 * d * c->esz > 256e6;
#define FM_PREFILL_GO(...) hipLaunchKernelGGL((k_prefill_kv<__VA_ARGS__>), dim3(c->pf_grid), dim3(256), PF_LDS_BYTES, c->stream, (const f16_t*)Xt, (const PrefillLayer*)c->pf_layers, seq_off, d / 32, d, D.M, c->pf_n)
#define FM_PREFILL(HDV)                                       \
  {                                                           \
    if (D.M % 256 || d % 256) FM_PREFILL_GO(HDV, true, false); \
    else if (past) FM_PREFILL_GO(HDV, false, true);           \
    else FM_PREFILL_GO(HDV, false, false);                    \
  }
    if (D.hd == 64) FM_PREFILL(64) else if (D.hd == 96) FM_PREFILL(96) else FM_PREFILL(128)
#undef FM_PREFILL
#undef FM_PREFILL_GO
  } else {
    float* kv = (float*)(Xt + (size_t)M32 * d);
    for (int st = 0; st < 5; st++)
      for (auto& L : c->stacks[st])
        for (int part = 0; part < parts; part++) {
          DecGemm a{};
          a.A = Xt; a.W = (const T*)L.ckv + (size_t)part * d * d; a.M = D.M; a.N = 2 * d / parts; a.KT = d / 32; a.Y = kv; a.ldy = a.N;
          dec_gemm<T, DE_F32, false>(a, 1, c->stream);
          const float *k = part == 0 ? kv : nullptr, *v = parts == 1 ? kv + d : part == 1 ? kv : nullptr;
#define FM_MEMKVH(HDV) hipLaunchKernelGGL((k_mem_kv_store<T, HDV>), dim3(D.M), dim3(256), 0, c->stream, k, v, a.N, (T*)L.Km + seq_off, (T*)L.Vm + seq_off, \
                                          D.H, D.M, (D.M + 31) / 32)
          if (D.hd == 64) FM_MEMKVH(64); else if (D.hd == 96) FM_MEMKVH(96); else FM_MEMKVH(128);
#undef FM_MEMKVH
        }
  }
  HIPCHK(c, hipGetLastError());
  return FM_OK;
}

// After a synchronisation: did the single-launch verify kernel give up waiting (it never hangs, it reports)?
// If so the passes enqueued since then have accepted nothing and committed nothing (k_accept / k_commit look at the
// same word), so the decode state is that of the last good commit.  The failure is reported once with its diagnosis,
// the words are re-armed, and the context continues on the per-operator path, which shares weights, caches and rings.
int check_persist(fm_ctx* c) {
  if (!c->persist) return FM_OK;
  unsigned w[9] = {0};
  HIPCHK(c, hipMemcpy(w, c->pk.abort_word, sizeof w, hipMemcpyDeviceToHost));
  if (!w[0]) return FM_OK;
  const unsigned rearm[9] = {0u, 0xFFFFFFFFu, 0u, 0u, 0u, 0u, 0u, 0u, 0u};
  HIPCHK(c, hipMemcpy(c->pk.abort_word, rearm, sizeof rearm, hipMemcpyHostToDevice));
  c->persist = false;
  drop_graphs(c);
  c->persist_failures++;
  return fail(c, FM_EHIP, "persistent verify kernel timed out: earliest stuck stage %u; first missing element: stage %u "
              "workgroup %u thread %u index %u expected tag %u saw %u; passes since then accepted nothing, the "
              "context continues with one launch per operator", w[1], w[5], w[6], w[7], w[8], w[3], w[4]);
}

// Build the parameter tables and the list of (blob range -> device destination) in manifest order.
int build_params(fm_ctx* c) {
  const Dims& D = c->D;
  const size_t d = D.d, ff = c->ff, hff = c->hff, V = D.V;
  size_t off = 0;
  auto item = [&](void* dst, size_t n, bool f32) { c->items.push_back({off, n, dst, f32, 0, 0, 0}); off += n; };
  // rope: leading rows that belong to queries or keys (half path: rotary pairs meet in one tile, see k_tile_weight)
  auto lin = [&](void* dst, size_t N, size_t K, size_t rope = 0) { c->items.push_back({off, N * K, dst, false, (int)N, (int)K, (int)rope}); off += N * K; };
  auto at = [&](void* base, size_t elems) { return (void*)((uint8_t*)base + elems * c->esz); };

  TRY(dalloc_t(c, &c->emb, V * d));
  item(c->emb, V * d, false);
  const int counts[5] = {c->cfg.l_cpre, c->cfg.l_vpre, c->cfg.l_face, c->cfg.l_vpost, c->cfg.l_cpost};
  for (int st = 0; st < 5; st++) {
    const int level = kStackLevel[st];
    const size_t cap = level_cap(c, level);
    for (int i = 0; i < counts[st]; i++) {
      Layer L{};
      L.level = level;
      TRY(dalloc(c, &L.g1, d)); TRY(dalloc(c, &L.g2, d)); TRY(dalloc(c, &L.g3, d));
      TRY(dalloc_t(c, &L.wqkv, 3 * d * d)); TRY(dalloc_t(c, &L.wo, d * d)); TRY(dalloc_t(c, &L.cq, d * d));
      TRY(dalloc_t(c, &L.ckv, 2 * d * d)); TRY(dalloc_t(c, &L.co, d * d));
      TRY(dalloc_t(c, &L.w1, ff * d)); TRY(dalloc_t(c, &L.w2, d * ff));
      TRY(dalloc_t(c, &L.Kc, D.S * cache_seq_elems(c, cap))); TRY(dalloc_t(c, &L.Vc, D.S * cache_seq_elems(c, cap)));
      TRY(dalloc_t(c, &L.Km, D.S * cache_seq_elems(c, D.M))); TRY(dalloc_t(c, &L.Vm, D.S * cache_seq_elems(c, D.M)));
      item(L.g1, d, true);
      lin(L.wqkv, 3 * d, d, 2 * d);   // wq, wk, wv are consecutive in the blob
      lin(L.wo, d, d);
      item(L.g2, d, true);
      lin(L.cq, d, d);
      lin(L.ckv, 2 * d, d);    // ck, cv consecutive
      lin(L.co, d, d);
      item(L.g3, d, true);
      lin(L.w1, ff, d);
      lin(L.w2, d, ff);
      c->stacks[st].push_back(L);
    }
  }
  TRY(dalloc_t(c, &c->short_cv, d * d)); lin(c->short_cv, d, d);
  TRY(dalloc_t(c, &c->short_vf, d * d)); lin(c->short_vf, d, d);
  TRY(dalloc(c, &c->gf, d)); item(c->gf, d, true);
  TRY(dalloc_t(c, &c->lm, (size_t)c->Vpad * d)); lin(c->lm, V, d);
  const int spcnt[3] = {D.Dc, D.nspv, D.nspf};
  // The heads of the three levels lie behind each other in device memory (point, face, coordinate: the order of the
  // merged row set), so that one grouped launch can serve all of them; the blob keeps its own order.
  {
    SpLevel& A = c->sp_all;
    A.cnt = D.Dc + D.nspv + D.nspf;
    const size_t n = A.cnt;
    TRY(dalloc(c, &A.g, n * d));
    TRY(dalloc_t(c, &A.wq, n * d * d)); TRY(dalloc_t(c, &A.wo, n * d * d)); TRY(dalloc_t(c, &A.cq, n * d * d));
    TRY(dalloc_t(c, &A.co, n * d * d)); TRY(dalloc_t(c, &A.lin, n * d * d));
    const size_t first[3] = {(size_t)D.nspv + D.nspf, 0, (size_t)D.nspv};
    for (int l = 0; l < 3; l++) {
      SpLevel& s = c->sp[l];
      s.g = A.g + first[l] * d;
      s.wq = at(A.wq, first[l] * d * d); s.wo = at(A.wo, first[l] * d * d); s.cq = at(A.cq, first[l] * d * d);
      s.co = at(A.co, first[l] * d * d); s.lin = at(A.lin, first[l] * d * d);
    }
  }
  for (int l = 0; l < 3; l++) {
    SpLevel& s = c->sp[l];
    s.cnt = spcnt[l];
    const size_t n = s.cnt;
    for (size_t k = 0; k < n; k++) {
      item(s.g + k * d, d, true);
      lin(at(s.wq, k * d * d), d, d, d); lin(at(s.wo, k * d * d), d, d);
      lin(at(s.cq, k * d * d), d, d); lin(at(s.co, k * d * d), d, d);
      lin(at(s.lin, k * d * d), d, d);
    }
  }
  HfLevel* hfs[2] = {&c->hfc, &c->hfv};
  const int hfcnt[2] = {D.nhfc, D.nhfv};
  for (int l = 0; l < 2; l++) {
    HfLevel& h = *hfs[l];
    h.cnt = hfcnt[l];
    const size_t n = h.cnt;
    TRY(dalloc(c, &h.g, n * d));
    TRY(dalloc_t(c, &h.wq, n * d * d)); TRY(dalloc_t(c, &h.w1, n * hff * d)); TRY(dalloc_t(c, &h.w2, n * d * hff));
    for (size_t k = 0; k < n; k++) {
      item(h.g + k * d, d, true);
      lin(at(h.wq, k * d * d), d, d, d);
      lin(at(h.w1, k * hff * d), hff, d);
      lin(at(h.w2, k * d * hff), d, hff);
    }
  }
  // label head of the correct stage (Sec. 3.2): [3][d], kept in fp32 (three dot products per point)
  TRY(dalloc(c, &c->label_w, 3 * d));
  item(c->label_w, 3 * d, true);
  c->blob_elems = off;
  return FM_OK;
}

// exchange buffers, stage records and argument block of the persistent verify kernel
int build_persist(fm_ctx* c) {
  const Dims& D = c->D;
  const size_t d = D.d;
  PkArgs& a = c->pk;
  memset(&a, 0, sizeof a);
  for (int st = 0; st < 5; st++) {
    a.first[st] = a.n_layers;
    a.count[st] = (int)c->stacks[st].size();
    a.n_layers += a.count[st];
    a.gain1[st] = (pk_cf_t)c->stacks[st][0].g1;
  }
  a.D = D; a.ff = c->ff; a.eps = c->cfg.rms_eps;
  a.R[0] = D.Bm; a.R[1] = D.VB; a.R[2] = D.FB;
  const int caps[3] = {D.capc, D.capv, D.capf};
  // splits of a head's keys: about one attention unit per workgroup, no more than there are groups of four blocks (one per wave),
  // as few as give the same longest walk, and no more parts than a merge takes in one trip to memory (16).  Steps in us, d = 1024 (16
  // heads) and d = 512 (8 heads): 16 splits 1966 / 836, 12 1972 / 859, 8 2022 / 871, 4 2238 / 919; 32 splits at d = 512, in two trips: 849
  auto splits = [&](int capb) {
    int ns = std::max(1, std::min(PK_NWG / D.H, PK_MAXSPLIT));
    if (const char* e = getenv("FM_PK_NSPLIT")) ns = std::max(1, std::min(atoi(e), PK_MAXSPLIT));       // measurement switch: splits per head
    const int groups = (capb + 3) / 4, rounds = (groups + ns - 1) / ns;
    return (groups + rounds - 1) / rounds;
  };
  for (int l = 0; l < 3; l++) {
    a.capb[l] = (caps[l] + 31) / 32;
    a.nsplit[l] = splits(a.capb[l]);
    a.pos[l] = (pk_ci_t)c->pos[l];
  }
  a.capbM = (D.M + 31) / 32;
  a.nsplitM = splits(a.capbM);
  a.vtok = (pk_ci_t)c->st.vtok;
  a.ring[0] = (pk_f_t)c->ring_hc; a.ring[1] = (pk_f_t)c->ring_hv; a.ring[2] = (pk_f_t)c->ring_yf; a.ring[3] = (pk_f_t)c->ring_yv;
  a.emb = (pk_cw_t)c->emb; a.logits = (pk_f_t)c->logits;
  const size_t nl = a.n_layers;
  // GEMM inputs (fp32 residual stream and its half-pair copy, attention outputs, FFN hidden): one region per layer,
  // so that no address is written twice within a launch
  // rows per exchange region: one group of 16, or two when the block is longer than 16 tokens
  a.RS = D.Bm > 16 ? 32 : 16;
  const size_t RS = a.RS, RH = RS / 2, RG = RS / 16;
  u64 *h[3], *x[3], *sq[3], *hT[4], *q[2], *att[2], *part[2], *mid;      // index 0: in front of the self-attention, 1: the cross-attention, 2: the FFN
  for (int i = 0; i < 3; i++) {
    const size_t n = nl + (i == 0);
    TRY(dalloc(c, &h[i], n * RS * d)); TRY(dalloc(c, &x[i], n * RH * d)); TRY(dalloc(c, &sq[i], n * RS * d / 16));
  }
  a.h = (pk_x_t)h[0]; a.x = (pk_x_t)x[0]; a.s = (pk_x_t)sq[0];
  for (int i = 0; i < 4; i++) { TRY(dalloc(c, &hT[i], RS * d)); a.hT[i] = (pk_x_t)hT[i]; }
  for (int i = 0; i < 2; i++) {      // queries (half pairs), attention outputs, parts of the splits
    TRY(dalloc(c, &q[i], RH * d)); TRY(dalloc(c, &att[i], nl * RH * d)); TRY(dalloc(c, &part[i], (size_t)D.H * PK_MAXSPLIT * RG * PK_PART));
  }
  TRY(dalloc(c, &a.pool, 2 * 8 * d)); TRY(dalloc(c, &mid, nl * RH * c->ff));
  TRY(dalloc(c, &a.newK, (size_t)D.H * RS * 32)); TRY(dalloc(c, &a.newV, (size_t)D.H * RS * 32));
  TRY(dalloc(c, &a.w2part, (d / 16) * RG * 3 * 256));
  {
    std::vector<PkRecord> recs;
    auto put = [&](std::initializer_list<const volatile void*> p) {
      PkRecord r{};
      int k = 0;
      for (const volatile void* v : p) r.p[k++] = (u64)v;
      recs.push_back(r);
    };
    float* ring[4] = {c->ring_hc, c->ring_hv, c->ring_yf, c->ring_yv};
    float* tap[3] = {c->tap_c, c->tap_v, c->tap_f};
    auto* newK = (u64*)a.newK;
    auto* newV = (u64*)a.newV;
    size_t l = 0;
    for (int st = 0; st < 5; st++) {
      const int lev = kStackLevel[st];
      for (size_t i = 0; i < c->stacks[st].size(); i++, l++) {
        const Layer& L = c->stacks[st][i];
        const bool last = i + 1 == c->stacks[st].size(), out = last && st < 4;      // a stack output feeds a level transition, not a norm
        auto H = [&](int k, size_t n) { return h[k] + n * RS * d; };
        auto X = [&](int k, size_t n) { return x[k] + n * RH * d; };
        auto Q = [&](int k, size_t n) { return sq[k] + n * RS * d / 16; };
        u64 *A0 = att[0] + l * RH * d, *A1 = att[1] + l * RH * d, *mi = mid + l * RH * c->ff;
        auto sizes = [](int ns, int capb) { return (const void*)(((u64)(unsigned)capb << 32) | (unsigned)ns); };
        put({L.wqkv, X(0, l), Q(0, l), L.Kc, q[0], newK, newV, c->cs[lev], L.Vc});
        put({L.Kc, L.Vc, q[0], part[0], A0, sizes(a.nsplit[lev], a.capb[lev]), (const void*)(u64)level_window(c, lev)});
        put({L.wo, A0, nullptr, H(0, l), H(1, l), X(1, l), Q(1, l), L.g2, last && st >= 2 ? tap[lev] : nullptr});
        put({L.cq, X(1, l), Q(1, l), nullptr, q[1]});
        put({L.Km, L.Vm, q[1], part[1], A1, sizes(a.nsplitM, a.capbM), nullptr});
        put({L.co, A1, nullptr, H(1, l), H(2, l), X(2, l), Q(2, l), L.g3, nullptr});
        put({L.w1, X(2, l), Q(2, l), nullptr, mi});
        put({L.w2, mi, nullptr, H(2, l), out ? hT[st] : H(0, l + 1), out ? nullptr : X(0, l + 1), Q(0, l + 1),
             last ? c->gf : c->stacks[st][i + 1].g1, out ? ring[st] : nullptr});
      }
    }
    for (int st = 0; st < 2; st++) {
      const size_t n = a.first[st + 1];
      put({st == 0 ? c->short_cv : c->short_vf, (u64*)a.pool + (size_t)st * 8 * d, nullptr, nullptr, h[0] + n * RS * d, x[0] + n * RH * d, sq[0] + n * RS * d / 16,
           c->stacks[st + 1][0].g1, nullptr});
    }
    put({c->lm, x[0] + nl * RH * d, sq[0] + nl * RS * d / 16});
    a.n_records = (int)recs.size();
    uint8_t* dev;
    TRY(dalloc(c, &dev, (recs.size() * sizeof(PkRecord) + 1023) / 1024 * 1024));
    if (hipMemcpy(dev, recs.data(), recs.size() * sizeof(PkRecord), hipMemcpyHostToDevice) != hipSuccess) return fail(c, FM_EHIP, "record table copy failed");
    a.records = (const PK_GLOBAL PkRecord*)dev;
  }
  TRY(dalloc(c, &a.abort_word, 16));
  if (hipMemset(a.abort_word + 1, 0xFF, 4) != hipSuccess) return fail(c, FM_EHIP, "hipMemset failed");
  a.run_flag = c->st.alive;
  if (const char* e = getenv("FM_PROFILE")) {
    if (e[0] == '1') TRY(dalloc(c, &a.prof, 1024));
    if (const char* ps = getenv("FM_PROFILE_STAGE")) a.prof_stage = atoi(ps); else a.prof_stage = -1;
  }
  TRY(dalloc(c, &c->pk_epoch, 1));
  a.epoch_word = c->pk_epoch;
  // test hooks for the bounded waits: a shorter bound, and an embedding that publishes under the wrong tag
  a.timeout_ticks = PK_TIMEOUT_TICKS;
  a.test_skew = 0;
  if (const char* e = getenv("FM_PK_TIMEOUT_TICKS")) a.timeout_ticks = strtoull(e, nullptr, 10);
  if (const char* e = getenv("FM_PK_TEST_SKEW")) a.test_skew = (unsigned)atoi(e);
  c->pk_lds = 0;   // the kernel uses static LDS only
  // all 256 workgroups must be resident at once: they wait for each other's results
  int dev = 0, cus = 0, per_cu = 0;
  if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, pk_kernel(a), 256, c->pk_lds) != hipSuccess ||
      (long)cus * per_cu < PK_NWG) {
    (void)hipGetLastError();
    c->persist = false;   // fall back to the per-launch path
  }
  return FM_OK;
}

int build_buffers(fm_ctx* c) {
  const Dims& D = c->D;
  const size_t d = D.d, S = D.S;
  StateDev& st = c->st;
  TRY(dalloc(c, &st.P, S)); TRY(dalloc(c, &st.main, S)); TRY(dalloc(c, &st.fin, S));
  TRY(dalloc(c, &st.firedv, S)); TRY(dalloc(c, &st.firedf, S));
  TRY(dalloc(c, &st.basec, S)); TRY(dalloc(c, &st.basev, S)); TRY(dalloc(c, &st.basef, S));
  TRY(dalloc(c, &st.vlen, S)); TRY(dalloc(c, &st.vtok, S * D.Bm)); TRY(dalloc(c, &st.y, S * D.Bm));
  TRY(dalloc(c, &st.hist, S * (D.maxtok + 1))); TRY(dalloc(c, &st.budget, 1)); TRY(dalloc(c, &st.alive, 1)); TRY(dalloc(c, &st.level_rows, 3));
  TRY(dalloc(c, &st.acc_hist, 3 * 32)); TRY(dalloc(c, &st.counters, 3)); TRY(dalloc(c, &st.kind, S));
  TRY(dalloc(c, &c->ring_hc, S * RS_C * d)); TRY(dalloc(c, &c->tap_c, S * RS_C * d));
  TRY(dalloc(c, &c->ring_hv, S * RS_V * d)); TRY(dalloc(c, &c->ring_yv, S * RS_V * d)); TRY(dalloc(c, &c->tap_v, S * RS_V * d));
  TRY(dalloc(c, &c->ring_yf, S * RS_F * d)); TRY(dalloc(c, &c->tap_f, S * RS_F * d));
  const size_t rows[3] = {(size_t)c->Rc, (size_t)c->Rv, (size_t)c->Rf};
  for (int l = 0; l < 3; l++) {
    TRY(dalloc(c, &c->pos[l], rows[l])); TRY(dalloc(c, &c->limx[l], rows[l]));
    TRY(dalloc(c, &c->cs[l], rows[l] * 64)); TRY(dalloc(c, &c->h[l], rows[l] * d));
    const size_t tiles = (rows[l] + 15) / 16;
    TRY(dalloc_t(c, &c->xg[l], tiles * 16 * d)); TRY(dalloc(c, &c->ssq[l], tiles * d));
  }
  {
    const size_t tiles = (rows[0] + 15) / 16;
    TRY(dalloc_t(c, &c->attX, tiles * 16 * d)); TRY(dalloc_t(c, &c->midX, tiles * 16 * c->ff));
    TRY(dalloc(c, &c->attn_arrived, (size_t)FM_ATTN_SETS * D.S * D.H));
    TRY(dalloc(c, &c->attn_ws, attn_ws_floats(D.H, D.S, FM_ATTN_SETS, D.hd)));
  }
  TRY(dalloc_t(c, &c->qT, rows[0] * d)); TRY(dalloc(c, &c->logits, rows[0] * D.V));
  // staging: conversion of the largest tensor, or the prefill (memory in T + fp32 K/V of one layer)
  size_t big = std::max((size_t)c->ff * d, (size_t)c->hff * d);
  big = std::max(big, 3 * d * d);
  big = std::max(big, (size_t)D.V * d);
  c->stage_elems = std::max(big, (size_t)(D.M + 31) / 32 * 32 * d + (size_t)D.M * 2 * d);
  TRY(dalloc(c, &c->stage, c->stage_elems));
  // draft rows
  const size_t nset[5] = {S * D.Dc, S * D.nspv, S * D.nspf, S * D.nhfv, S * 2 * D.nhfc};
  size_t maxset = 1;
  for (int i = 3; i < 5; i++) {
    maxset = std::max(maxset, nset[i]);
    TRY(dalloc(c, (const float***)&c->dr.src[i], nset[i]));
    TRY(dalloc(c, &c->dr.lim[i], nset[i])); TRY(dalloc(c, &c->dr.limx[i], nset[i]));
    TRY(dalloc(c, &c->dr.cs[i], nset[i] * 64));
  }
  const int G_all = D.Dc + D.nspv + D.nspf;
  {
    // One table for the three SP row sets: rows [sequence][point heads | face heads | coordinate heads], as the heads lie in
    // memory, so that a grouped launch over all heads sees S rows per head with one stride.
    const size_t nsp = nset[0] + nset[1] + nset[2], np = (size_t)D.hd / 2;
    maxset = std::max(maxset, nsp);
    const float** src; int *lim, *limx; float2* cs;
    TRY(dalloc(c, (const float***)&src, nsp)); TRY(dalloc(c, &lim, nsp)); TRY(dalloc(c, &limx, nsp));
    TRY(dalloc(c, &cs, nsp * 64));
    const size_t first[3] = {(size_t)D.nspv + D.nspf, 0, (size_t)D.nspv};
    for (int i = 0; i < 5; i++) c->dr.rs[i] = i < 3 ? G_all : i == 3 ? D.nhfv : 2 * D.nhfc;
    for (int i = 0; i < 3; i++) {
      c->dr.src[i] = src + first[i]; c->dr.lim[i] = lim + first[i];
      c->dr.limx[i] = limx + first[i]; c->dr.cs[i] = cs + first[i] * np;
    }
  }
  TRY(dalloc(c, &c->dr.alive, S)); TRY(dalloc(c, &c->dr.firev, S)); TRY(dalloc(c, &c->dr.firef, S)); TRY(dalloc(c, &c->dr.flags, 2));
  TRY(dalloc(c, &c->hfv_out, nset[3] * d));
  const size_t nLM = S * (D.Dc + 2 * D.nhfc);
  // Outputs of the SP heads: one buffer [sequence][point | face | coordinate heads][d].  The output head reads its rows
  // (coordinate SP heads of every sequence, then the coordinate HF rows) through a pointer table.
  TRY(dalloc(c, &c->dh, nLM * d));
  TRY(dalloc(c, &c->spv_out, (size_t)S * std::max(G_all, 1) * d));
  c->spf_out = c->spv_out + (size_t)D.nspv * d;
  {
    std::vector<const float*> tab(std::max<size_t>(nLM, 1));
    for (size_t i = 0; i < nLM; i++)
      tab[i] = i < S * (size_t)D.Dc ? c->spv_out + ((i / D.Dc) * G_all + D.nspv + D.nspf + i % D.Dc) * d : c->dh + i * d;
    TRY(dalloc(c, (const float***)&c->lm_src, tab.size()));
    HIPCHK(c, hipMemcpy(c->lm_src, tab.data(), tab.size() * sizeof(float*), hipMemcpyHostToDevice));
  }
  TRY(dalloc(c, &c->dlogits, nLM * D.V));
  const size_t rmax = std::max(maxset, nLM);
  TRY(dalloc_t(c, &c->dq, rmax * d));
  {
    c->sp_tiles = (int)(S + 15) / 16; c->hf_tiles[0] = (int)(S + 15) / 16; c->hf_tiles[1] = (int)(2 * S + 15) / 16;
    const size_t sp = (size_t)G_all * c->sp_tiles, hv = (size_t)D.nhfv * c->hf_tiles[0], hc = (size_t)D.nhfc * c->hf_tiles[1], lmt = (nLM + 15) / 16;
    TRY(dalloc_t(c, &c->dX, std::max(std::max(sp, hv), std::max(std::max(hc, lmt), (size_t)1)) * 16 * d));
    TRY(dalloc_t(c, &c->dmidX, std::max(std::max(sp * d, std::max(hv, hc) * c->hff), (size_t)1) * 16));
  }
  TRY(dalloc(c, &c->dist_c, S * std::max(D.Dc, 1) * D.V));
  TRY(dalloc(c, &c->dist_v, S * std::max(D.nhfc, 1) * D.V)); TRY(dalloc(c, &c->dist_f, S * std::max(D.nhfc, 1) * D.V));
  TRY(dalloc(c, &c->lab_v, S * std::max(D.nspv, 1) * 3)); TRY(dalloc(c, &c->lab_f, S * std::max(D.nhfv, 1) * 3));
  TRY(dalloc(c, &c->params_dev, 1)); TRY(dalloc(c, &c->commits_dev, 1));
  c->smp = Sampling{c->params_dev, nullptr, nullptr, nullptr, nullptr};
  TRY(dalloc(c, &c->smp.qrow, S * D.Bm * D.V)); TRY(dalloc(c, &c->smp.qsum, S * D.Bm));
  TRY(dalloc(c, &c->smp.qtok, S * D.Bm)); TRY(dalloc(c, &c->smp.accflag, S * D.Bm));
  c->db = DraftBufs{c->tap_c, c->tap_v, c->tap_f, c->ring_yf, c->spv_out, c->spf_out, c->hfv_out, G_all, G_all};
  TRY(dalloc(c, &c->gen_tok, S * D.Bm)); TRY(dalloc(c, &c->gen_len, S)); TRY(dalloc(c, &c->gen_acc, S));
  if (c->persist) TRY(build_persist(c));
  if (c->bf16) {
    if (d >= 128) {            // one launch for all blocks; narrower models: one GEMM and one scatter launch per block
      std::vector<PrefillLayer> tab;
      for (int st = 0; st < 5; st++)
        for (auto& L : c->stacks[st]) tab.push_back(PrefillLayer{(const f16_t*)L.ckv, (f16_t*)L.Km, (f16_t*)L.Vm});
      uint8_t* raw = nullptr;
      TRY(dalloc(c, &raw, tab.size() * sizeof(PrefillLayer)));
      c->pf_layers = (PrefillLayer*)raw;
      HIPCHK(c, hipMemcpy(c->pf_layers, tab.data(), tab.size() * sizeof(PrefillLayer), hipMemcpyHostToDevice));
      c->pf_n = (int)tab.size();
#define FM_PREFILL_LDS(HDV, ...) HIPCHK(c, hipFuncSetAttribute((const void*)k_prefill_kv<HDV, __VA_ARGS__>, hipFuncAttributeMaxDynamicSharedMemorySize, PF_LDS_BYTES))
#define FM_PREFILL_ALL(HDV) FM_PREFILL_LDS(HDV, false, false); FM_PREFILL_LDS(HDV, false, true); FM_PREFILL_LDS(HDV, true, false)
      FM_PREFILL_ALL(64); FM_PREFILL_ALL(96); FM_PREFILL_ALL(128);
#undef FM_PREFILL_ALL
#undef FM_PREFILL_LDS
      hipDeviceProp_t prop;
      int dev = 0;
      HIPCHK(c, hipGetDevice(&dev));
      HIPCHK(c, hipGetDeviceProperties(&prop, dev));
      c->pf_grid = std::max(8, prop.multiProcessorCount / 8 * 8);
    }
  }
  if (hipHostMalloc((void**)&c->prog, sizeof(Progress)) != hipSuccess || hipHostMalloc((void**)&c->host_counts, 99 * sizeof(unsigned long long)) != hipSuccess)
    return fail(c, FM_ENOMEM, "hipHostMalloc failed");
  memset(c->prog, 0, sizeof(Progress));
  for (int i = 0; i < fm_ctx::E_COUNT; i++) HIPCHK(c, hipEventCreate(&c->ev[i]));
  // The launches of the fp32 path and of narrow half-precision models are shorter than the host needs to enqueue one (d = 256, 3 sequences: 18.9
  // ms a mesh as launches, 15.6 as graphs); from about d = 768 there is no difference, and the single-launch verify kernel leaves
  // few launches (medium model, one sequence: 2055 us as launches, 2071 us as two graphs).
  const char* ge = getenv("FM_GRAPH");          // "0" / "1": never / always (measurement switch)
  c->graphs_on = ge ? ge[0] != '0' : !c->bf16 || (!c->persist && D.d <= 512);
  return FM_OK;
}

}  // namespace

// ------------------------------------------------------------------------------------------
// C ABI
// ------------------------------------------------------------------------------------------
extern "C" {

int fm_create(const fm_config* cfg, void* hip_stream, fm_ctx** out) {
  if (!cfg || !out) return FM_EINVAL;
  *out = nullptr;
  const fm_config& g = *cfg;
  if (g.d_model <= 0 || g.n_heads <= 0 || g.d_model % g.n_heads != 0) return FM_EINVAL;
  const int hd = g.d_model / g.n_heads;          // 64, or the paper's own widths 96 and 128
  if (hd != 64 && hd != 96 && hd != 128) return FM_EINVAL;
  if (g.ffn_mult < 1 || g.hf_ffn_mult < 1 || g.n_bins < 1 || g.mem_len < 1) return FM_EINVAL;
  if (g.l_cpre < 1 || g.l_cpost < 1 || g.l_vpre < 1 || g.l_vpost < 1 || g.l_face < 1) return FM_EINVAL;
  if (g.dtype != FM_DTYPE_F32 && g.dtype != FM_DTYPE_BF16) return FM_EINVAL;
  if (g.max_batch < 1 || g.max_batch > 64 || g.max_tokens < 9 || g.max_tokens % 9 != 0) return FM_EINVAL;
  if (g.draft_coord < 0 || g.draft_point < 0 || g.draft_face < 0) return FM_EINVAL;
  if (g.draft_point % 3 != 0 || g.draft_face % 9 != 0) return FM_EINVAL;
  if ((g.draft_point > 0 || g.draft_face > 0) && g.draft_coord < 2 && !(g.rules_off & 2)) return FM_EINVAL;  // rule (B) leaves 3 tokens to the coordinate level
  const int Bm = std::max(std::max(1 + g.draft_coord, g.draft_point), std::max(g.draft_face, 1));
  if (Bm > 27) return FM_EINVAL;  // rings hold 32 coordinate positions: block + 2 carried rows
  if (!(g.rope_base > 1.f) || !(g.rms_eps > 0.f)) return FM_EINVAL;
  if (g.window < 0 || g.window % 9 != 0) return FM_EINVAL;
  if (g.rules_off & ~3) return FM_EINVAL;

  fm_ctx* c = new (std::nothrow) fm_ctx();
  if (!c) return FM_ENOMEM;
  c->cfg = g;
  c->stream = (hipStream_t)hip_stream;
  c->bf16 = g.dtype == FM_DTYPE_BF16;
  c->esz = c->bf16 ? 2 : 4;
  c->ff = g.ffn_mult * g.d_model;
  c->hff = g.hf_ffn_mult * g.d_model;
  Dims& D = c->D;
  D.d = g.d_model; D.H = g.n_heads; D.hd = hd; D.V = g.n_bins + 3; D.S = g.max_batch; D.Bm = Bm;
  D.VB = (Bm + 2) / 3; D.FB = (Bm + 8) / 9; D.M = g.mem_len;
  D.maxtok = g.max_tokens;
  D.capc = g.max_tokens; D.capv = (g.max_tokens + 2) / 3 + 1; D.capf = (g.max_tokens + 8) / 9 + 1;
  D.wc = D.wv = D.wf = 0;
  if (g.window > 0 && g.window < g.max_tokens) {
    // rings: the window plus the rows of one pass (a rejected block leaves stale rows behind the committed
    // length; they must only ever overwrite positions that no later query can see), in groups of four 32-key
    // blocks (the rows of one pass then never meet twice in the blocks one wave of an attention range walks)
    D.wc = g.window; D.wv = g.window / 3; D.wf = g.window / 9;
    auto ring = [](int w, int rows) { return (w + rows + 2 + 127) / 128 * 128; };
    D.capc = ring(D.wc, D.Bm); D.capv = ring(D.wv, D.VB); D.capf = ring(D.wf, D.FB);
  }
  D.Dc = g.draft_coord; D.m = g.draft_point; D.n = g.draft_face;
  D.nspv = std::max(D.m / 3 - 1, 0); D.nspf = std::max(D.n / 9 - 1, 0);
  D.t0 = (g.rules_off & 2) ? 0 : 3; D.j0 = (g.rules_off & 2) ? 0 : 1;
  D.nhfc = std::max(std::max(D.m, D.n) - D.t0, 0); D.nhfv = std::max(D.n / 3 - D.j0, 0);
  D.ruleA = (g.rules_off & 1) ? 0 : 1;
  D.nbins = g.n_bins; D.ban = g.ban_specials ? 1 : 0; D.eos = g.n_bins + 1; D.pad = g.n_bins + 2;
  c->Vpad = (D.V + 63) / 64 * 64;
  c->Rc = D.S * D.Bm; c->Rv = D.S * D.VB; c->Rf = D.S * D.FB;
  for (int i = 0; i < 64; i++) c->inv.v[i] = std::pow((double)g.rope_base, -(double)i / (hd / 2.0));
  c->weights_loaded = false;
  c->prefilled.assign(D.S, false);
  {
    const int nl = g.l_cpre + g.l_cpost + g.l_vpre + g.l_vpost + g.l_face;
    const char* env = getenv("FM_PERSIST");
    // (a wave of the single-launch kernel holds 8 K fragments of a quarter of the hidden width: up to 4096)
    c->persist = c->bf16 && D.hd == 64 && D.S == 1 && D.Bm <= 32 && D.d % 128 == 0 && D.d <= 1024 && c->ff % 512 == 0 && c->ff <= 4096 && nl < 62 &&
                 !(env && env[0] == '0');
  }
  int rc = build_params(c);
  if (rc == FM_OK) rc = build_buffers(c);
  if (rc == FM_OK) {
    // this GPU's copy of the static staging array: address looked up once per device, with that device current
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) rc = fail(c, FM_EHIP, "hipGetDevice failed");
    else {
      std::lock_guard<std::mutex> lk(g_scratch_mu);
      if (!g_scratch_addr[dev]) {
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) rc = fail(c, FM_EHIP, "hipGetSymbolAddress(scratch) failed: %s", hipGetErrorString(e));
        else g_scratch_addr[dev] = p;
      }
      c->static_scratch = (unsigned char*)g_scratch_addr[dev];
    }
  }
  if (rc == FM_OK) {
    const int budget = g.max_tokens;
    if (hipMemcpy(c->st.budget, &budget, sizeof(int), hipMemcpyHostToDevice) != hipSuccess) rc = FM_EHIP;
    // all sequences start finished until they are prefilled
    std::vector<int> ones(D.S, 1);
    if (hipMemcpy(c->st.fin, ones.data(), sizeof(int) * D.S, hipMemcpyHostToDevice) != hipSuccess) rc = FM_EHIP;
  }
  if (rc != FM_OK) {
    fprintf(stderr, "fm_create: %s\n", c->err.c_str());
    release(c);
    return rc;
  }
  // algorithmic weight bytes of one verify pass
  const double d2 = (double)D.d * D.d;
  const int nl = g.l_cpre + g.l_cpost + g.l_vpre + g.l_vpost + g.l_face;
  c->weight_bytes = c->esz * (nl * (6.0 + 2.0 * g.ffn_mult) * d2 + 2.0 * d2 + (double)D.V * D.d);
  *out = c;
  return FM_OK;
}

int fm_destroy(fm_ctx* c) {
  if (!c) return FM_EINVAL;
  (void)hipStreamSynchronize(c->stream);
  release(c);
  return FM_OK;
}

const char* fm_last_error(const fm_ctx* c) { return c ? c->err.c_str() : "null context"; }
int32_t fm_block_max(const fm_ctx* c) { return c ? c->D.Bm : FM_EINVAL; }
int32_t fm_verify_path(const fm_ctx* c) { return c ? (c->persist ? 1 : 0) : FM_EINVAL; }
int64_t fm_blob_elems(const fm_ctx* c) { return c ? (int64_t)c->blob_elems : FM_EINVAL; }

int fm_load_weights(fm_ctx* c, const float* blob, size_t n_floats) {
  if (!c) return FM_EINVAL;
  if (!blob) return fail(c, FM_EINVAL, "null blob");
  if (n_floats != c->blob_elems) return fail(c, FM_EINVAL, "blob has %zu floats, expected %zu", n_floats, c->blob_elems);
  for (const LoadItem& it : c->items) {
    size_t done = 0;
    while (done < it.n) {
      const size_t n = std::min(it.n - done, c->stage_elems);
      if (it.f32) {
        HIPCHK(c, hipMemcpyAsync((float*)it.dst + done, blob + it.blob_off + done, n * 4, hipMemcpyHostToDevice, c->stream));
      } else {
        HIPCHK(c, hipMemcpyAsync(c->stage, blob + it.blob_off + done, n * 4, hipMemcpyHostToDevice, c->stream));
        if (it.N > 0) {
          if (n != it.n) return fail(c, FM_EINVAL, "staging buffer smaller than a weight matrix");
          const int Npad = (it.N + 15) / 16 * 16;
          if (c->bf16) hipLaunchKernelGGL((k_tile_weight<f16_t>), dim3(1024), dim3(256), 0, c->stream, c->stage, (f16_t*)it.dst, it.N, it.K, Npad, it.rope, c->D.hd);
          else hipLaunchKernelGGL((k_tile_weight<float>), dim3(1024), dim3(256), 0, c->stream, c->stage, (float*)it.dst, it.N, it.K, Npad, it.rope, c->D.hd);
        } else if (c->bf16)
          hipLaunchKernelGGL((k_convert<f16_t>), dim3(1024), dim3(256), 0, c->stream, c->stage, (f16_t*)it.dst + done, (long)n);
        else
          hipLaunchKernelGGL((k_convert<float>), dim3(1024), dim3(256), 0, c->stream, c->stage, (float*)it.dst + done, (long)n);
      }
      HIPCHK(c, hipStreamSynchronize(c->stream));  // the staging buffer is reused
      done += n;
    }
  }
  HIPCHK(c, hipGetLastError());
  c->weights_loaded = true;
  return FM_OK;
}

int fm_prefill_condition(fm_ctx* c, int32_t seq, const float* mem_dev) {
  if (!c) return FM_EINVAL;
  if (!c->weights_loaded) return fail(c, FM_ESTATE, "weights not loaded");
  if (seq < 0 || seq >= c->D.S) return fail(c, FM_EINVAL, "sequence %d out of range [0,%d)", seq, c->D.S);
  if (!mem_dev) return fail(c, FM_EINVAL, "null condition memory");
  const size_t room = c->stage_elems * sizeof(float);
  int rc = c->bf16 ? prefill_impl<f16_t>(c, seq, mem_dev, c->stage, room) : prefill_impl<float>(c, seq, mem_dev, c->stage, room);
  if (rc == FM_OK) c->prefilled[seq] = true;
  return rc;
}

int fm_prefill_condition_static(fm_ctx* c, int32_t seq, const float* mem_dev) {
  if (!c) return FM_EINVAL;
  if (!c->weights_loaded) return fail(c, FM_ESTATE, "weights not loaded");
  if (seq < 0 || seq >= c->D.S) return fail(c, FM_EINVAL, "sequence %d out of range [0,%d)", seq, c->D.S);
  if (!mem_dev) return fail(c, FM_EINVAL, "null condition memory");
  if (!c->static_scratch) return fail(c, FM_ESTATE, "no static staging area on this device");
  const size_t need = prefill_stage_bytes(c);
  if (need > FM_STATIC_SCRATCH_BYTES)
    return fail(c, FM_EINVAL, "condition memory of %d x %d needs %zu staging bytes, the static area holds %u: use fm_prefill_condition",
                c->D.M, c->D.d, need, (unsigned)FM_STATIC_SCRATCH_BYTES);
  int rc = c->bf16 ? prefill_impl<f16_t>(c, seq, mem_dev, c->static_scratch, FM_STATIC_SCRATCH_BYTES)
                   : prefill_impl<float>(c, seq, mem_dev, c->static_scratch, FM_STATIC_SCRATCH_BYTES);
  if (rc == FM_OK) c->prefilled[seq] = true;
  return rc;
}

int fm_draft(fm_ctx* c, int32_t* block_tok, int32_t* block_len) {
  if (!c) return FM_EINVAL;
  if (!c->weights_loaded) return fail(c, FM_ESTATE, "weights not loaded");
  if (!block_tok || !block_len) return fail(c, FM_EINVAL, "null block buffer");
  const int rc = run_graphed(c, fm_ctx::GraphKey{G_DRAFT, step_flags(c, 1), c->correct_hist, {block_tok, block_len, nullptr, nullptr}}, false,
                             [&] { return draft_any(c, block_tok, block_len, 1); });
  return rc == FM_OK && c->sticky_error ? FM_EINVAL : rc;
}

int fm_set_sampling(fm_ctx* c, float temperature, uint64_t seed) {
  if (!c) return FM_EINVAL;
  if (!(temperature >= 0.f) || temperature > 1e4f) return fail(c, FM_EINVAL, "temperature %g outside [0, 1e4]", (double)temperature);
  c->params.temperature = temperature;
  c->params.seed = seed;
  return put_params(c);
}

int fm_set_correct(fm_ctx* c, int32_t hist_vertices) {
  if (!c) return FM_EINVAL;
  if (hist_vertices < 0) return fail(c, FM_EINVAL, "hist_vertices %d < 0", hist_vertices);
  c->correct_hist = hist_vertices;
  return FM_OK;
}

int fm_correct(fm_ctx* c, int32_t* block_tok, const int32_t* block_len, int32_t* labels_out) {
  if (!c) return FM_EINVAL;
  if (!c->weights_loaded) return fail(c, FM_ESTATE, "weights not loaded");
  if (c->correct_hist <= 0) return fail(c, FM_ESTATE, "correct stage is off: call fm_set_correct before the fm_draft whose block is corrected");
  if (!block_tok || !block_len) return fail(c, FM_EINVAL, "null block buffer");
  hipLaunchKernelGGL(k_correct, dim3(c->D.S), dim3(64), 0, c->stream, c->st, c->D, c->lab_v, c->lab_f, c->correct_hist,
                     block_tok, block_len, labels_out);
  HIPCHK(c, hipGetLastError());
  return FM_OK;
}

int fm_verify_block(fm_ctx* c, const int32_t* block_tok, const int32_t* block_len, float* logits, int32_t* accepted) {
  if (!c) return FM_EINVAL;
  if (!c->weights_loaded) return fail(c, FM_ESTATE, "weights not loaded");
  if (!block_tok || !block_len || !accepted) return fail(c, FM_EINVAL, "null block / accepted buffer");
  const int rc = run_graphed(c, fm_ctx::GraphKey{G_VERIFY, step_flags(c, 1), c->correct_hist, {block_tok, block_len, logits, accepted}}, false,
                             [&] { return verify_any(c, block_tok, block_len, logits, accepted); });
  return rc == FM_OK && c->sticky_error ? FM_EINVAL : rc;
}

int fm_commit(fm_ctx* c, const int32_t* accepted) {
  if (!c) return FM_EINVAL;
  if (!accepted) return fail(c, FM_EINVAL, "null accepted buffer");
  return commit_any(c, accepted, false);
}

int fm_set_budget(fm_ctx* c, int32_t max_faces) {
  if (!c) return FM_EINVAL;
  if (max_faces < 1 || 9 * max_faces > c->D.maxtok) return fail(c, FM_EINVAL, "max_faces %d outside [1,%d]", max_faces, c->D.maxtok / 9);
  hipLaunchKernelGGL(k_set_budget, dim3(1), dim3(64), 0, c->stream, c->st, c->D, 9 * max_faces, 0u, c->commits_dev);
  HIPCHK(c, hipGetLastError());
  return FM_OK;
}

int fm_set_draft_replay(fm_ctx* c, const int32_t* stream_dev, int32_t stride, int32_t n_valid, float keep_prob, uint64_t seed) {
  if (!c) return FM_EINVAL;
  if (stream_dev && (stride < n_valid || n_valid < 0 || !(keep_prob >= 0.f && keep_prob <= 1.f)))
    return fail(c, FM_EINVAL, "bad replay arguments");
  c->params.replay = Replay{stream_dev, stride, n_valid, keep_prob, (unsigned long long)seed};
  return put_params(c);
}

int fm_read_state(fm_ctx* c, int32_t* host_out) {
  if (!c || !host_out) return FM_EINVAL;
  const int S = c->D.S;
  std::vector<int> P(S), mn(S), fin(S);
  HIPCHK(c, hipStreamSynchronize(c->stream));
  HIPCHK(c, hipMemcpy(P.data(), c->st.P, S * 4, hipMemcpyDeviceToHost));
  HIPCHK(c, hipMemcpy(mn.data(), c->st.main, S * 4, hipMemcpyDeviceToHost));
  HIPCHK(c, hipMemcpy(fin.data(), c->st.fin, S * 4, hipMemcpyDeviceToHost));
  TRY(check_persist(c));
  for (int s = 0; s < S; s++) {
    host_out[s * 6 + 0] = P[s];
    host_out[s * 6 + 1] = (P[s] + 2) / 3;
    host_out[s * 6 + 2] = (P[s] + 8) / 9;
    host_out[s * 6 + 3] = mn[s];
    host_out[s * 6 + 4] = fin[s];
    host_out[s * 6 + 5] = P[s];
  }
  return FM_OK;
}

int fm_debug_profile(fm_ctx* c, uint64_t* host_out, int32_t n) {
  if (!c || !host_out || n < 1 || n > 1024) return FM_EINVAL;
  if (!c->persist || !c->pk.prof) return fail(c, FM_ESTATE, "stage profiling is off (FM_PROFILE=1 at fm_create, persistent path only)");
  HIPCHK(c, hipStreamSynchronize(c->stream));
  HIPCHK(c, hipMemcpy(host_out, c->pk.prof, (size_t)n * 8, hipMemcpyDeviceToHost));
  std::vector<unsigned long long> init(1024, 0ull);
  init[0] = ~0ull;
  HIPCHK(c, hipMemcpy(c->pk.prof, init.data(), 1024 * 8, hipMemcpyHostToDevice));   // re-arm
  return FM_OK;
}

int fm_debug_draft(fm_ctx* c, int32_t which, float* host_out) {
  if (!c) return FM_EINVAL;
  const Dims& D = c->D;
  if (which == -1 || which == -2) { c->params.keep_rows = which == -1 ? 1 : 0; return put_params(c); }
  if (!host_out) return fail(c, FM_EINVAL, "null output");
  const float* src = which == 0 ? c->smp.qrow : which == 1 ? c->lab_v : which == 2 ? c->lab_f : nullptr;
  if (!src) return fail(c, FM_EINVAL, "draft buffer %d out of range", which);
  const size_t n = which == 0 ? (size_t)D.S * D.Bm * D.V : which == 1 ? (size_t)D.S * std::max(D.nspv, 1) * 3 : (size_t)D.S * std::max(D.nhfv, 1) * 3;
  HIPCHK(c, hipStreamSynchronize(c->stream));
  HIPCHK(c, hipMemcpy(host_out, src, n * sizeof(float), hipMemcpyDeviceToHost));
  return FM_OK;
}

int fm_debug_ring(fm_ctx* c, int32_t which, float* host_out) {
  if (!c || !host_out) return FM_EINVAL;
  float* src[7] = {c->ring_hc, c->ring_hv, c->ring_yf, c->ring_yv, c->tap_c, c->tap_v, c->tap_f};
  const int rs[7] = {RS_C, RS_V, RS_F, RS_V, RS_C, RS_V, RS_F};
  if (which < 0 || which >= 7) return fail(c, FM_EINVAL, "ring %d out of range", which);
  HIPCHK(c, hipStreamSynchronize(c->stream));
  HIPCHK(c, hipMemcpy(host_out, src[which], (size_t)c->D.S * rs[which] * c->D.d * sizeof(float), hipMemcpyDeviceToHost));
  return FM_OK;
}

int fm_debug_mem_kv(fm_ctx* c, int32_t seq, int32_t block, float* host_k, float* host_v) {
  if (!c || !host_k || !host_v) return FM_EINVAL;
  if (seq < 0 || seq >= c->D.S) return fail(c, FM_EINVAL, "sequence %d out of range", seq);
  if (!c->prefilled[seq]) return fail(c, FM_ESTATE, "sequence %d has no condition memory", seq);
  const Layer* L = nullptr;
  int left = block;
  for (int st = 0; st < 5 && !L && left >= 0; st++) {
    if (left < (int)c->stacks[st].size()) L = &c->stacks[st][left];
    else left -= (int)c->stacks[st].size();
  }
  if (block < 0 || !L) return fail(c, FM_EINVAL, "block %d out of range", block);
  const Dims& D = c->D;
  const size_t n = cache_seq_elems(c, D.M);
  std::vector<unsigned char> raw(n * c->esz);
  HIPCHK(c, hipStreamSynchronize(c->stream));
  for (int kv = 0; kv < 2; kv++) {
    const unsigned char* src = (const unsigned char*)(kv ? L->Vm : L->Km) + (size_t)seq * n * c->esz;
    HIPCHK(c, hipMemcpy(raw.data(), src, raw.size(), hipMemcpyDeviceToHost));
    float* out = kv ? host_v : host_k;
    const int hd = D.hd, capb = (D.M + 31) / 32;
    for (int m = 0; m < D.M; m++)
      for (int i = 0; i < D.d; i++) {
        const int hh = i / hd, e = i % hd;
        // the blocked layouts: 32-key blocks of a head; K in MFMA fragment order, V as [dim][key slot]
        const int r = m & 31;
        size_t o = ((size_t)hh * capb + (m >> 5)) * 32 * hd;
        if (kv == 0) o += (size_t)((((r >> 4) * (hd / 32) + (e >> 5)) * 64 + (r & 15) + 16 * ((e & 31) >> 3)) * 8 + (e & 7));
        else o += (size_t)e * 32 + ((r & 15) >> 2) * 8 + (r >> 4) * 4 + (r & 3);
        out[(size_t)m * D.d + i] = c->bf16 ? (float)((const f16_t*)raw.data())[o] : ((const float*)raw.data())[o];
      }
  }
  return FM_OK;
}

int fm_verify_bytes(fm_ctx* c, double* host_bytes) {
  if (!c || !host_bytes) return FM_EINVAL;
  const int S = c->D.S;
  std::vector<int> P(S), fin(S);
  HIPCHK(c, hipStreamSynchronize(c->stream));
  HIPCHK(c, hipMemcpy(P.data(), c->st.P, S * 4, hipMemcpyDeviceToHost));
  HIPCHK(c, hipMemcpy(fin.data(), c->st.fin, S * 4, hipMemcpyDeviceToHost));
  double bytes = c->weight_bytes;
  const fm_config& g = c->cfg;
  for (int s = 0; s < S; s++) {
    if (fin[s]) continue;
    double Lc = P[s], Lv = (P[s] + 2) / 3, Lf = (P[s] + 8) / 9;
    const double M = c->D.M;
    if (c->D.wc > 0) { Lc = std::min<double>(Lc, c->D.wc); Lv = std::min<double>(Lv, c->D.wv); Lf = std::min<double>(Lf, c->D.wf); }
    bytes += c->esz * 2.0 * c->D.d *
             ((g.l_cpre + g.l_cpost) * (Lc + M) + (g.l_vpre + g.l_vpost) * (Lv + M) + g.l_face * (Lf + M));
  }
  *host_bytes = bytes;
  return FM_OK;
}

int fm_measure_peaks(fm_ctx* c, double* host_out) {
  if (!c || !host_out) return FM_EINVAL;
  const size_t bytes = (size_t)1 << 30;
  float4 *a = nullptr, *b = nullptr;
  float* sink = nullptr;
  hipEvent_t e0 = nullptr, e1 = nullptr;
  int rc = FM_OK;
  auto cleanup = [&]() {
    if (a) (void)hipFree(a);
    if (b) (void)hipFree(b);
    if (sink) (void)hipFree(sink);
    if (e0) (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
  };
#define PK_TRY(x) do { if ((x) != hipSuccess) { (void)hipGetLastError(); cleanup(); return fail(c, FM_EHIP, "peak probe: %s failed", #x); } } while (0)
  PK_TRY(hipStreamSynchronize(c->stream));
  PK_TRY(hipMalloc((void**)&a, bytes)); PK_TRY(hipMalloc((void**)&b, bytes)); PK_TRY(hipMalloc((void**)&sink, 1024 * 256 * 4));
  PK_TRY(hipMemsetAsync(a, 0, bytes, c->stream)); PK_TRY(hipMemsetAsync(b, 0, bytes, c->stream));
  PK_TRY(hipEventCreate(&e0)); PK_TRY(hipEventCreate(&e1));
  const long n16 = (long)(bytes / 16);
  const int reps = 5, iters = 4000, wgs = 1024;
  float ms = 0.f;
  // streaming read
  hipLaunchKernelGGL(k_probe_read, dim3(2048), dim3(256), 0, c->stream, a, sink, n16);
  PK_TRY(hipEventRecord(e0, c->stream));
  for (int i = 0; i < reps; i++) hipLaunchKernelGGL(k_probe_read, dim3(2048), dim3(256), 0, c->stream, a, sink, n16);
  PK_TRY(hipEventRecord(e1, c->stream)); PK_TRY(hipEventSynchronize(e1)); PK_TRY(hipEventElapsedTime(&ms, e0, e1));
  host_out[0] = (double)bytes * reps / (ms * 1e-3) / 1e9;
  // streaming copy (read + write bytes)
  hipLaunchKernelGGL(k_probe_copy, dim3(32768), dim3(256), 0, c->stream, a, b, n16);
  PK_TRY(hipEventRecord(e0, c->stream));
  for (int i = 0; i < reps; i++) hipLaunchKernelGGL(k_probe_copy, dim3(32768), dim3(256), 0, c->stream, a, b, n16);
  PK_TRY(hipEventRecord(e1, c->stream)); PK_TRY(hipEventSynchronize(e1)); PK_TRY(hipEventElapsedTime(&ms, e0, e1));
  host_out[1] = 2.0 * (double)bytes * reps / (ms * 1e-3) / 1e9;
  // MFMA loop
  hipLaunchKernelGGL(k_probe_mfma, dim3(wgs), dim3(256), 0, c->stream, sink, 100);
  PK_TRY(hipEventRecord(e0, c->stream));
  hipLaunchKernelGGL(k_probe_mfma, dim3(wgs), dim3(256), 0, c->stream, sink, iters);
  PK_TRY(hipEventRecord(e1, c->stream)); PK_TRY(hipEventSynchronize(e1)); PK_TRY(hipEventElapsedTime(&ms, e0, e1));
  host_out[2] = 2.0 * 32 * 32 * 16 * 8.0 * iters * 4.0 * wgs / (ms * 1e-3) / 1e12;
#undef PK_TRY
  cleanup();
  return rc;
}

int fm_measure_exchange(fm_ctx* c, int32_t workgroups, int32_t bytes, int32_t pingpong, double* host_out) {
  if (!c || !host_out) return FM_EINVAL;
  if (workgroups < 2 || workgroups > 256 || bytes < workgroups * 8 || bytes > 49152 || bytes % (workgroups * 16) != 0)
    return fail(c, FM_EINVAL, "exchange probe: 2..256 workgroups, bytes a multiple of 16 per workgroup, at most 49152");
  int dev = 0, cus = 0, per_cu = 0;
  if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
      hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k_probe_exchange, 256, 0) != hipSuccess || (long)cus * per_cu < workgroups) {
    (void)hipGetLastError();
    return fail(c, FM_ESTATE, "exchange probe: %d workgroups cannot be resident together on this device", workgroups);
  }
  const int vol = bytes / 8, nstage = 2000;
  unsigned long long *buf = nullptr, *ticks = nullptr;
  unsigned* words = nullptr;
  auto cleanup = [&]() {
    if (buf) (void)hipFree(buf);
    if (ticks) (void)hipFree(ticks);
    if (words) (void)hipFree(words);
  };
#define PK_TRY(x) do { if ((x) != hipSuccess) { (void)hipGetLastError(); cleanup(); return fail(c, FM_EHIP, "exchange probe: %s failed", #x); } } while (0)
  PK_TRY(hipStreamSynchronize(c->stream));
  PK_TRY(hipMalloc((void**)&buf, (size_t)3 * vol * 8)); PK_TRY(hipMalloc((void**)&ticks, 16)); PK_TRY(hipMalloc((void**)&words, 256));
  PK_TRY(hipMemsetAsync(buf, 0, (size_t)3 * vol * 8, c->stream)); PK_TRY(hipMemsetAsync(ticks, 0, 16, c->stream));
  PK_TRY(hipMemsetAsync(words, 0, 256, c->stream));
  hipLaunchKernelGGL(k_probe_exchange, dim3(workgroups), dim3(256), 0, c->stream, buf, words, words + 32, ticks, vol, nstage, pingpong ? 1 : 0);
  PK_TRY(hipStreamSynchronize(c->stream));
  unsigned long long t[2] = {0, 0};
  unsigned ab = 0;
  PK_TRY(hipMemcpy(t, ticks, 16, hipMemcpyDeviceToHost)); PK_TRY(hipMemcpy(&ab, words + 32, 4, hipMemcpyDeviceToHost));
#undef PK_TRY
  cleanup();
  if (ab) return fail(c, FM_EHIP, "exchange probe: a bounded wait expired");
  host_out[0] = (double)(t[1] - t[0]) * 0.01 / nstage;       // microseconds per round (100 MHz wall clock)
  return FM_OK;
}

int fm_measure_gemm(fm_ctx* c, int32_t rows, double* host_out) {
  if (!c || !host_out) return FM_EINVAL;
  if (!c->bf16 || !c->weights_loaded) return fail(c, FM_ESTATE, "GEMM probe needs the half-precision path with weights loaded");
  if (rows < 1 || rows > 65536) return fail(c, FM_EINVAL, "rows %d outside [1, 65536]", rows);
  const int d = c->D.d, N = c->ff;
  const Layer& L = c->stacks[0][0];
  f16_t *X = nullptr, *Y = nullptr;
  hipEvent_t e0 = nullptr, e1 = nullptr;
  auto cleanup = [&]() {
    if (X) (void)hipFree(X);
    if (Y) (void)hipFree(Y);
    if (e0) (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
  };
#define PK_TRY(x) do { if ((x) != hipSuccess) { (void)hipGetLastError(); cleanup(); return fail(c, FM_EHIP, "GEMM probe: %s failed", #x); } } while (0)
  PK_TRY(hipStreamSynchronize(c->stream));
  const size_t prow = (size_t)(rows + 15) / 16 * 16;
  PK_TRY(hipMalloc((void**)&X, prow * d * 2)); PK_TRY(hipMalloc((void**)&Y, prow * N * 2));
  PK_TRY(hipMemsetAsync(X, 0, prow * d * 2, c->stream));
  PK_TRY(hipEventCreate(&e0)); PK_TRY(hipEventCreate(&e1));
  // Y[rows, ff] = gelu(X[rows, d] W1^T): the FFN up projection of the first block, half in and out
  DecGemm a{};
  a.A = X; a.W = (const f16_t*)L.w1; a.M = rows; a.N = N; a.KT = d / 32; a.X = Y;
  const int reps = rows <= 256 ? 50 : 10;
  float ms = 0.f;
  // FM_GEMM_PROBE_CYCLE = n: successive launches walk the up projections of n different blocks (n x 8 d^2 bytes
  // of weights), which tells a last-level-cache hit from an L2 hit from HBM
  std::vector<const void*> ws;
  for (int st = 0; st < 5; st++) for (auto& Lx : c->stacks[st]) ws.push_back(Lx.w1);
  int cyc = 1;
  if (const char* e = getenv("FM_GEMM_PROBE_CYCLE")) cyc = std::max(1, std::min(atoi(e), (int)ws.size()));
  for (int i = 0; i < cyc; i++) { a.W = ws[i]; dec_gemm<f16_t, DE_GELU, false>(a, 1, c->stream); }
  PK_TRY(hipEventRecord(e0, c->stream));
  for (int i = 0; i < reps; i++) { a.W = ws[i % cyc]; dec_gemm<f16_t, DE_GELU, false>(a, 1, c->stream); }
  PK_TRY(hipEventRecord(e1, c->stream)); PK_TRY(hipEventSynchronize(e1)); PK_TRY(hipEventElapsedTime(&ms, e0, e1));
  host_out[0] = ms / reps;
  host_out[1] = 2.0 * rows * (double)N * d * reps / (ms * 1e-3) / 1e12;
#undef PK_TRY
  cleanup();
  return FM_OK;
}

int fm_generate(fm_ctx* c, int32_t max_faces, int32_t speculative, int32_t* out_tok, int32_t* out_len, fm_stats* stats) {
  if (!c) return FM_EINVAL;
  if (!c->weights_loaded) return fail(c, FM_ESTATE, "weights not loaded");
  if (!out_tok || !out_len) return fail(c, FM_EINVAL, "null output buffer");
  for (int s = 0; s < c->D.S; s++)
    if (!c->prefilled[s]) return fail(c, FM_ESTATE, "sequence %d has no condition memory", s);
  if (max_faces < 1 || 9 * max_faces > c->D.maxtok) return fail(c, FM_EINVAL, "max_faces %d outside [1,%d]", max_faces, c->D.maxtok / 9);
  const Dims& D = c->D;
  c->generation = c->generation % 0xFFFu + 1;
  hipLaunchKernelGGL(k_set_budget, dim3(1), dim3(64), 0, c->stream, c->st, D, 9 * max_faces, c->generation, c->commits_dev);
  HIPCHK(c, hipGetLastError());
  HIPCHK(c, hipEventRecord(c->ev[fm_ctx::E_BEGIN], c->stream));
  const int flags = step_flags(c, speculative), hist = c->correct_hist;
  const int per_step = speculative ? D.Bm : 1;         // most tokens a step can commit
  auto draft = [&]() -> int {
    TRY(draft_any(c, c->gen_tok, c->gen_len, speculative));
    return speculative && c->correct_hist > 0 ? fm_correct(c, c->gen_tok, c->gen_len, nullptr) : FM_OK;
  };
  auto verify = [&]() -> int { return verify_any(c, c->gen_tok, c->gen_len, nullptr, c->gen_acc); };
  // A step in as few launches as it takes: without drafts the block is the main token (k_verify_setup knows it), one sequence is committed by the
  // launch that chooses.
  auto whole = [&]() -> int {
    if (speculative) TRY(draft());
    return verify_any(c, speculative ? c->gen_tok : nullptr, speculative ? c->gen_len : nullptr, nullptr, c->gen_acc, true);
  };
  const fm_ctx::GraphKey kd{G_DRAFT, flags, hist, {c->gen_tok, c->gen_len, c->gen_acc, c}}, kv{G_VERIFY, flags, hist, {c->gen_tok, c->gen_len, nullptr, c->gen_acc}},
      ks{G_STEP, flags, hist, {c->gen_tok, c->gen_len, nullptr, c->gen_acc}};
  const int sample_every = 32;
  const long max_steps = 9L * max_faces + 1 + 128;     // + the steps a failed pass of the single-launch kernel may void
  bool phase_pending = false;
  long phase_samples = 0;
  double ms_phase[3] = {0.0, 0.0, 0.0};
  auto take_phases = [&]() -> int {
    float a = 0.f, b = 0.f, d = 0.f;
    HIPCHK(c, hipEventElapsedTime(&a, c->ev[fm_ctx::E_P0], c->ev[fm_ctx::E_P1]));
    HIPCHK(c, hipEventElapsedTime(&b, c->ev[fm_ctx::E_P1], c->ev[fm_ctx::E_P2]));
    HIPCHK(c, hipEventElapsedTime(&d, c->ev[fm_ctx::E_P2], c->ev[fm_ctx::E_P3]));
    ms_phase[0] += a; ms_phase[1] += b; ms_phase[2] += d;
    phase_samples++;
    phase_pending = false;
    return FM_OK;
  };
  // what the device has reported: steps committed by every sequence, and per sequence its length then (-1 = finished)
  long done = 0;
  bool alive = true, failed = false;
  int len[64];
  auto look = [&]() {
    unsigned least = FM_COMMIT_MASK;
    alive = failed = false;
    for (int s = 0; s < D.S; s++) {
      const unsigned long long w = __atomic_load_n(&c->prog->seq[s], __ATOMIC_RELAXED);
      const unsigned gen = progress_call(w), v = progress_state(w);
      const unsigned ahead = gen == c->generation ? progress_ahead(w, done) : 0u;      // commits since `done`
      least = std::min(least, ahead);
      len[s] = gen != c->generation ? 0 : v == 1 ? -1 : (int)v - 2;
      if (done + ahead > 0 && v == 0) failed = true;
      if (done + ahead == 0 || len[s] != -1) alive = true;
    }
    done += least;
  };
  int rc = FM_OK;
  for (long step = 0; step < max_steps; step++) {
    // The device must never wait for the host, and no step must run for nothing.  A further step is enqueued at once while it
    // cannot be the one after the last: some sequence stays below its budget even if all that is enqueued is accepted whole (where
    // EOS may be emitted: one step more than the device has finished).  Else only when the device has finished what it has.
    // While steps are queued behind the one that runs the thread sleeps between looks (20 us, about 75 with the scheduler's slack: no step is
    // as short); only for the last steps of a mesh, each of which the device would wait behind, does it look all the time.
    for (unsigned looks = 1;; looks++) {
      look();
      const long ahead = step - done;              // steps enqueued and not yet committed
      if (ahead == 0 || (done > 0 && (failed || !alive))) break;
      if (!D.ban && ahead < 2) break;
      if (D.ban && done > 0 && ahead < 6) {
        bool sure = false;
        for (int s = 0; s < D.S; s++) sure |= len[s] >= 0 && len[s] + per_step * ahead < 9L * max_faces;
        if (sure) break;
      }
      if (looks % 512 == 0) {
        const hipError_t q = hipStreamQuery(c->stream);
        if (q != hipSuccess && q != hipErrorNotReady) return fail(c, FM_EHIP, "decode loop: %s", hipGetErrorString(q));
        (void)hipGetLastError();
        if (q == hipSuccess) {
          look();
          if (step - done > 0) return fail(c, FM_EHIP, "decode loop: the stream is idle but %ld steps were not reported", step - done);
        }
      }
      if (ahead > 1) {
        std::this_thread::sleep_for(std::chrono::microseconds(20));
        continue;
      }
#if defined(__x86_64__)
      for (int i = 0; i < 8; i++) __builtin_ia32_pause();
#endif
    }
    if (done > 0 && failed) {
      // the single-launch verify kernel gave up in some pass: nothing was accepted or committed since, so the loop
      // simply goes on with one launch per operator (message kept in fm_last_error)
      HIPCHK(c, hipStreamSynchronize(c->stream));
      (void)check_persist(c);
    } else if (done > 0 && !alive) {
      break;
    }
    // one step per interval carries the phase marks, once the marks of the previous sample have been read
    bool sample = step % sample_every == 1;
    if (sample && phase_pending) {
      if (hipEventQuery(c->ev[fm_ctx::E_P3]) == hipSuccess) TRY(take_phases());
      else { (void)hipGetLastError(); sample = false; }
    }
    if (sample) {
      HIPCHK(c, hipEventRecord(c->ev[fm_ctx::E_P0], c->stream));
      rc = run_graphed(c, kd, true, draft);
      if (rc == FM_OK) {
        HIPCHK(c, hipEventRecord(c->ev[fm_ctx::E_P1], c->stream));
        rc = run_graphed(c, kv, true, verify);
      }
      if (rc == FM_OK) {
        HIPCHK(c, hipEventRecord(c->ev[fm_ctx::E_P2], c->stream));
        rc = commit_any(c, c->gen_acc, true);
      }
      if (rc == FM_OK) { HIPCHK(c, hipEventRecord(c->ev[fm_ctx::E_P3], c->stream)); phase_pending = true; }
    } else {
      rc = run_graphed(c, ks, true, whole);
    }
    if (rc == FM_OK && c->sticky_error) rc = FM_EINVAL;
    if (rc != FM_OK) return rc;
  }
  HIPCHK(c, hipEventRecord(c->ev[fm_ctx::E_END], c->stream));
  hipLaunchKernelGGL(k_finish, dim3(std::min(32, (D.maxtok + 255) / 256), D.S), dim3(256), 0, c->stream, c->st, D, out_tok, out_len, c->host_counts);
  HIPCHK(c, hipGetLastError());
  HIPCHK(c, hipStreamSynchronize(c->stream));
  TRY(check_persist(c));      // a failure in the very last step: reported, the caller may call again
  if (phase_pending) TRY(take_phases());
  if (stats) {
    const unsigned long long *cnt = c->host_counts, *acc = c->host_counts + 3;
    float ms = 0.f;
    HIPCHK(c, hipEventElapsedTime(&ms, c->ev[fm_ctx::E_BEGIN], c->ev[fm_ctx::E_END]));
    stats->steps = (int64_t)cnt[0];
    stats->tokens = (int64_t)cnt[1];
    for (int k = 0; k < 3; k++)
      for (int i = 0; i < 32; i++) stats->acc_hist[k][i] = (int64_t)acc[k * 32 + i];
    stats->ms_total = ms;
    const double n = phase_samples > 0 ? (double)phase_samples : 1.0;
    stats->ms_draft = ms_phase[0] / n; stats->ms_verify = ms_phase[1] / n; stats->ms_commit = ms_phase[2] / n;
    stats->phase_samples = phase_samples;
    stats->nonfinite_rows = (int64_t)cnt[2];
  }
  return FM_OK;
}

}  // extern "C"
