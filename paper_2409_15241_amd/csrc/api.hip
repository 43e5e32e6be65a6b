// Host side of the C ABI declared in include/domino.h: argument validation, memory layout of the
// saved / workspace blocks, the p x q piece schedule over the caller's stream pool (one block, one
// block cut at its all-reduce points, or a stack of blocks whose row groups run on without joining),
// and the single-kernel entry points.  No device memory is allocated here and no host synchronisation
// is performed by the layer calls.
#include "../../include/domino.h"

#include <hip/hip_runtime.h>

#include <atomic>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <initializer_list>
#include <map>
#include <mutex>
#include <vector>

#include "attention.h"
#include "eltwise.h"
#include "gemm.h"
#include "norm.h"
#include "probe.h"

namespace {

thread_local char g_err[512] = "";

int fail(int code, const char* fmt, ...) {
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(g_err, sizeof(g_err), fmt, ap);
  va_end(ap);
  return code;
}
int fail_hip(hipError_t e, const char* what) {
  return fail(DOMINO_ERR_HIP, "%s: %s", what, hipGetErrorString(e));
}
#define HIP_TRY(expr, what)                                  \
  do {                                                       \
    hipError_t e_ = (expr);                                  \
    if (e_ != hipSuccess) return fail_hip(e_, what);         \
  } while (0)

// One-time notes about conditions that do not change results but cost time (process-wide, see domino_last_warning).
std::mutex g_warn_mutex;
char g_warn[512] = "";
bool g_warned_queues = false;

// Streams that share a hardware queue run one after the other.  The HIP runtime reads GPU_MAX_HW_QUEUES once, when it
// starts (default 4, one of which serves the null stream), so all the library can do is look at the environment the
// process was started with and say what it sees.  `used`: the streams that a call puts launches on, at most three of its pool.
void note_hw_queues(int used) {
  if (used < 2) return;
  std::lock_guard<std::mutex> lock(g_warn_mutex);
  if (g_warned_queues) return;
  const char* env = getenv("GPU_MAX_HW_QUEUES");
  if ((env ? atoi(env) : 4) >= used + 1) return;
  g_warned_queues = true;
  snprintf(g_warn, sizeof(g_warn),
           "a call uses %d streams of its pool side by side, but GPU_MAX_HW_QUEUES is %s: with fewer hardware queues than these "
           "streams and the null stream some of them share a queue and run one after the other; set GPU_MAX_HW_QUEUES >= %d "
           "before the HIP runtime starts", used, env ? env : "unset (runtime default 4)", used + 1);
}

constexpr size_t ALIGN = 256;
size_t align_up(size_t v) { return (v + ALIGN - 1) / ALIGN * ALIGN; }
constexpr long TWO_GIB = 1L << 31;

// ---------------------------------------------------------------------------------- layout
struct Layout {
  int h, n, t, r, p, q, b, s, f, d, nl, hl, fl, upc, M, Ms, hq;
  bool llama;
  bool merged;       // weight and vector gradients of a block in one launch each over all slices (see merged_wgrads)
  bool per_slice;    // cfg->wgrad_per_slice
  bool beside;       // the backward's weight gradients run on a stream of their own (see wgrads_beside)
  int groups;        // row groups: consecutive slices whose launches are one launch each (see row_groups)
  // saved block (bytes)
  size_t ln1, qkv, ctx, lse, x1, ln2, pre, act, mean1, rstd1, mean2, rstd2, saved_total;
  // workspace block (bytes)
  size_t d_pre, dx1, dctx, dqkv, dot, red, wpart, ws_total;
  int wsplits;       // contraction ranges of the weight gradients' one launch, whose sums meet in wpart
  // partial column sums: area k starts area_off[k] floats in and holds, for every slice (the norms') or row group (the
  // column sums'), area_rows[k] rows of area_n[k] floats; red_floats = size of all areas
  size_t red_floats, area_off[8];
  int area_rows[8], area_n[8];

  size_t area(int k, int i) const { return area_off[k] + (size_t)i * area_rows[k] * area_n[k]; }     // of slice or group i
  int first_slice(int g) const { return (int)((long)p * g / groups); }      // group g = slices [first_slice(g), first_slice(g + 1))
};

enum { AREA_G1 = 0, AREA_B1, AREA_G2, AREA_B2, AREA_BQKV, AREA_BO, AREA_BUP, AREA_BDOWN, NAREAS };

// Two rules say how a call spreads over its streams.  Both look at the block alone, so neither the arithmetic nor a bit
// of any result depends on the stream pool, and the parts of one backward agree on the layout of what they hand on.
// In 256x256 tiles of the four weight gradients and of a product as wide as the block:
int tiles256(long m, long n) { return (int)((m + 255) / 256 * ((n + 255) / 256)); }
int wgrad_tiles(const Layout& l) { return tiles256(l.fl, l.h) + tiles256(l.h, l.upc) + tiles256(l.hl, l.h) + tiles256(l.h, 3 * l.hl); }

// The backward's weight gradients run on a stream of their own where their tiles fill most of the 256 compute units or
// more: then they fill what the chain of input gradients, attention and norms leaves idle.  Below that they follow on the
// chain's stream as one launch, which has the chip to itself (forward + backward without and with the side stream, us:
// 24000 tokens of a 1536-wide shard, 114 tiles, 1656 and 1950; GPT-3 2.7B, 160 tiles, 1464 and 1703; a 3072-wide Llama
// shard of 4096 tokens, 228 tiles, 547 and 574; Llama-2 7B, 400 tiles, 2048 tokens, 486 and 491, 8192 tokens, 1421 and 1384,
// 16384 tokens, 2658 and 2571; 13B, 620 tiles, 2048 tokens, 703 and 652, 8192 tokens, 2129 and 2019).  The second stream also costs a
// call about 100 us of host time (event records and waits) and 5 to 10 us at each of its edges on the GPU, whatever the
// block's size: blocks under 40 GFLOP of weight gradients (13B's at 512 tokens) keep to one.
bool wgrads_beside(const Layout& l) {
  return wgrad_tiles(l) > 200 && 2.0 * l.M * l.h * (4.0 * l.hl + l.upc + l.fl) >= 40e9;
}

// Row slices cut the batch so that a program can reduce one slice's partial sums over the ranks while the next slice
// computes.  Inside one library call nothing waits for a single slice, so consecutive slices are launched together, as
// one launch over the rows of all of them: larger launches fill 256 compute units better, and a step of many small
// launches pays for the launches.  What the slices' streams used to buy, two chains of dependent launches side by side
// so that one fills the chip while the other drains, needs two groups and no more (four streams share the four hardware
// queues that a process gets by default, and slices that meet on a queue run one after the other), and only pays in
// wide blocks where a group's launches fill the chip on their own (two groups and one beside a side stream, us: Llama-2 7B
// with 16384 tokens, 1024 tiles, 2571 and 2691; with 8192, 512 tiles, 1384 and 1415; with 4096, 256 tiles, 823 and 781; 13B with
// 4096 tokens, 320 tiles, 1134 and 1062; with 2048, 765 and 653.  13B with 8192 tokens, 640 tiles, 2030 and 2061, four such
// blocks in a stack 7980 and 8150, one in parts 2132 and 2078; 30B, 896 tiles, 3521 and 3542, forward 1242 and 1254; Llama-2 13B with 16384,
// 1280 tiles, 4172 and 4234.)
int row_groups(const Layout& l) { return l.p > 2 && wgrads_beside(l) && tiles256(l.M, l.h) >= 512 ? 2 : 1; }

int validate(const domino_cfg* c, Layout* L) {
  if (!c) return fail(DOMINO_ERR_NULL_POINTER, "cfg is NULL");
  if (c->hidden <= 0 || c->heads <= 0 || c->tp <= 0 || c->p <= 0 || c->q <= 0 || c->batch <= 0 ||
      c->seq <= 0 || c->ffn <= 0)
    return fail(DOMINO_ERR_INVALID_ARG, "hidden, heads, tp, p, q, batch, seq, ffn must be positive");
  if (c->rank < 0 || c->rank >= c->tp) return fail(DOMINO_ERR_INVALID_ARG, "rank %d outside [0, tp=%d)", c->rank, c->tp);
  if (c->arch != DOMINO_ARCH_GPT && c->arch != DOMINO_ARCH_LLAMA)
    return fail(DOMINO_ERR_INVALID_ARG, "arch %d is neither GPT (0) nor Llama (1)", c->arch);
  if (!(c->norm_eps > 0.0f) || !(c->norm_eps < 1.0f)) return fail(DOMINO_ERR_INVALID_ARG, "norm_eps must lie in (0, 1)");
  if (c->arch == DOMINO_ARCH_LLAMA && !(c->rope_base > 1.0f)) return fail(DOMINO_ERR_INVALID_ARG, "rope_base must exceed 1");
  if (c->hidden % c->heads) return fail(DOMINO_ERR_INDIVISIBLE, "hidden %d %% heads %d != 0", c->hidden, c->heads);
  if (c->heads % c->tp) return fail(DOMINO_ERR_INDIVISIBLE, "heads %d %% tp %d != 0", c->heads, c->tp);
  if (c->ffn % c->tp) return fail(DOMINO_ERR_INDIVISIBLE, "ffn %d %% tp %d != 0", c->ffn, c->tp);
  if (c->batch % c->p) return fail(DOMINO_ERR_INDIVISIBLE, "batch %d %% p %d != 0", c->batch, c->p);
  if (c->hidden % c->q) return fail(DOMINO_ERR_INDIVISIBLE, "hidden %d %% q %d != 0", c->hidden, c->q);
  Layout l{};
  l.h = c->hidden; l.n = c->heads; l.t = c->tp; l.r = c->rank; l.p = c->p; l.q = c->q;
  l.b = c->batch; l.s = c->seq; l.f = c->ffn;
  l.llama = c->arch == DOMINO_ARCH_LLAMA;
  if (c->wgrad_per_slice != 0 && c->wgrad_per_slice != 1) return fail(DOMINO_ERR_INVALID_ARG, "wgrad_per_slice must be 0 or 1");
  l.merged = c->p > 2 && !c->wgrad_per_slice;
  l.per_slice = c->wgrad_per_slice;
  l.d = l.h / l.n; l.nl = l.n / l.t; l.hl = l.nl * l.d; l.fl = l.f / l.t;
  l.upc = l.fl * (l.llama ? 2 : 1);
  l.hq = l.h / l.q;
  if (l.d != 64 && l.d != 80 && l.d != 128) return fail(DOMINO_ERR_UNSUPPORTED, "head_dim %d not in {64, 80, 128}", l.d);
  if (l.h % 8 || l.hq % 8 || l.fl % 8) return fail(DOMINO_ERR_UNSUPPORTED, "hidden, hidden/q and ffn/tp must be multiples of 8");
  if (l.llama && l.fl % 32) return fail(DOMINO_ERR_UNSUPPORTED, "SwiGLU needs ffn/tp to be a multiple of 32");
  if (l.h > 8192) return fail(DOMINO_ERR_UNSUPPORTED, "hidden %d exceeds 8192", l.h);
  const long M = (long)l.b * l.s;
  long widest = l.h;
  if (3 * l.hl > widest) widest = 3 * l.hl;
  if (l.upc > widest) widest = l.upc;
  if (M * widest * 2 >= TWO_GIB) return fail(DOMINO_ERR_UNSUPPORTED, "an activation tensor would reach 2 GiB");
  if ((long)l.h * widest * 4 >= TWO_GIB) return fail(DOMINO_ERR_UNSUPPORTED, "a weight-gradient tensor would reach 2 GiB");
  l.M = (int)M;
  l.Ms = l.M / l.p;
  l.beside = wgrads_beside(l);
  l.groups = row_groups(l);

  size_t o = 0;
  auto take = [&](size_t bytes) { size_t at = o; o += align_up(bytes); return at; };
  const size_t Mz = (size_t)l.M;
  l.ln1 = take(Mz * l.h * 2);
  l.qkv = take(Mz * 3 * l.hl * 2);
  l.ctx = take(Mz * l.hl * 2);
  l.lse = take((size_t)l.b * l.nl * l.s * 4);
  l.x1 = take(Mz * l.h * 2);
  l.ln2 = take(Mz * l.h * 2);
  l.pre = take(Mz * l.upc * 2);
  l.act = take(Mz * l.fl * 2);
  l.mean1 = take(Mz * 4); l.rstd1 = take(Mz * 4); l.mean2 = take(Mz * 4); l.rstd2 = take(Mz * 4);
  l.saved_total = o;

  o = 0;
  l.d_pre = take(Mz * l.upc * 2);
  l.dx1 = take(Mz * l.h * 2);
  l.dctx = take(Mz * l.hl * 2);
  l.dqkv = take(Mz * 3 * l.hl * 2);
  l.dot = take((size_t)l.b * l.nl * l.s * 4);
  {
    const int nb = norm_bwd_slice_blocks((l.p + l.groups - 1) / l.groups, l.Ms, l.h);
    // b_o and b_down come out of the Norm2 backward kernel (one partial row per workgroup), the others from column-sum passes
    const int rows[NAREAS] = {nb, nb, nb, nb, COLSUM_PARTS, nb, COLSUM_PARTS, nb};
    const int width[NAREAS] = {l.h, l.h, l.h, l.h, 3 * l.hl, l.h, l.fl, l.h};
    size_t fo = 0;
    for (int k = 0; k < NAREAS; ++k) {
      l.area_off[k] = fo; l.area_rows[k] = rows[k]; l.area_n[k] = width[k];
      fo += (size_t)rows[k] * width[k] * (k == AREA_BQKV || k == AREA_BUP ? l.groups : l.p);
    }
    l.red_floats = (fo + 63) / 64 * 64;
  }
  l.red = take(l.red_floats * 4);
  const long wfloats = (long)l.h * (4L * l.hl + l.upc + l.fl);
  l.wsplits = l.beside || l.per_slice ? 1 : gemm_wgrad_splits(wgrad_tiles(l), l.M, wfloats);
  l.wpart = take(l.wsplits > 1 ? (size_t)wfloats * 4 * l.wsplits : 0);
  l.ws_total = o;
  if (L) *L = l;
  return DOMINO_OK;
}

// ---------------------------------------------------------------------------------- events, profiling
std::mutex g_mutex;
// Events for the cross-stream edges of a call (timing disabled), kept per device and handed out again from the
// first by the next call on that device: an edge already enqueued keeps the record it was made with.
struct EventPool { std::vector<hipEvent_t> events; size_t used = 0; };
std::map<int, EventPool> g_pools;
EventPool* g_pool = nullptr;               // the current device's pool, set by begin_call()

// Pools under which a layer or stack call has been replayed from a HIP graph bit for bit: 1, 2 or 4 streams, with
// 1, 2 or 4 of them carrying slices.  Instantiating a graph captured with a pool of 3 or 8 streams has aborted
// inside the runtime; until the reason is known such captures are refused before anything is enqueued.
bool capture_pool_ok(int nstreams, int p) {
  const int nslice = p < nstreams ? p : nstreams;
  auto ok = [](int v) { return v == 1 || v == 2 || v == 4; };
  return ok(nstreams) && ok(nslice);
}

thread_local bool g_capturing = false;     // streams[0] of the call being enqueued is under HIP graph capture

int begin_call(void* const* streams, int nstreams, int p) {
  int dev = 0;
  HIP_TRY(hipGetDevice(&dev), "hipGetDevice");
  g_pool = &g_pools[dev];
  t_tail.open = false;                       // (a call that failed half way may have left it)
  hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
  HIP_TRY(hipStreamIsCapturing(static_cast<hipStream_t>(streams[0]), &cs), "hipStreamIsCapturing");
  g_capturing = cs != hipStreamCaptureStatusNone;
  if (g_capturing) {
    if (!capture_pool_ok(nstreams, p))
      return fail(DOMINO_ERR_UNSUPPORTED, "streams[0] is being captured into a HIP graph with a pool of %d streams for %d row "
                  "slices: capture is supported for pools of 1, 2 or 4 streams only (see domino_capture_supported)", nstreams, p);
    // every edge of one capture keeps an event of its own: the calls recorded into a capture (a forward and a
    // backward, say) never re-record an event that an earlier call of the same capture recorded
  } else {
    g_pool->used = 0;
  }
  return DOMINO_OK;
}

// The events order streams of one device and are never looked at from the host, so they go without the fence that would make
// the work before them visible there and to other devices (a program's own event, synchronisation or copy behind the call on streams[0]
// has its own): a record then holds its stream up for 5 us and
// not for 6 to 8 (forward + backward, us, with and without the fence: 13B with 2048 tokens 655 and 641, with 8192 2042 and 2028, in parts 2124 and
// 2115; Llama-2 7B level).
int next_sync_event(hipEvent_t* ev) {
  if (g_pool->used == g_pool->events.size()) {
    hipEvent_t e;
    HIP_TRY(hipEventCreateWithFlags(&e, hipEventDisableTiming | hipEventDisableSystemFence), "hipEventCreate");
    g_pool->events.push_back(e);
  }
  *ev = g_pool->events[g_pool->used++];
  return DOMINO_OK;
}

// residual_out: the block output as a pass of its own; in the MLP-down product's epilogue it is part of gemm_down
enum ProfClass {
  PC_NORM_FWD = 0, PC_GEMM_QKV, PC_ROPE, PC_ATTN_FWD, PC_GEMM_OUT, PC_GEMM_UP, PC_GEMM_DOWN, PC_RESID_OUT,
  PC_DGRAD_DOWN, PC_WGRAD_DOWN, PC_DGRAD_UP, PC_WGRAD_UP, PC_NORM_BWD, PC_DGRAD_OUT, PC_WGRAD_OUT,
  PC_ATTN_BWD, PC_DGRAD_QKV, PC_WGRAD_QKV, PC_COLSUM, PC_WGRAD_JOINED, PC_COUNT
};
const char* const PROF_NAMES[PC_COUNT] = {
  "norm_fwd", "gemm_qkv", "rope", "attn_fwd", "gemm_out", "gemm_up", "gemm_down", "residual_out",
  "dgrad_down", "wgrad_down", "dgrad_up", "wgrad_up", "norm_bwd", "dgrad_out", "wgrad_out",
  "attn_bwd", "dgrad_qkv", "wgrad_qkv", "colsum", "wgrad_joined"};

std::atomic<bool> g_prof_on{false};      // per-launch timing (domino_profile_enable): adds event records to a call, changes none of its launches
struct ProfRec { int cls; hipStream_t stream; hipEvent_t start, stop; };
std::vector<ProfRec> g_prof_recs;
std::vector<hipEvent_t> g_prof_free;

int prof_event(hipEvent_t* ev) {
  if (!g_prof_free.empty()) { *ev = g_prof_free.back(); g_prof_free.pop_back(); return DOMINO_OK; }
  HIP_TRY(hipEventCreate(ev), "hipEventCreate");
  return DOMINO_OK;
}

// RAII bracket around the launches of one step on one stream; launches = false: the step only hands work over to a later
// launch (GemmArgs::join, ColsumJobs::join, HeldTail), which has the bracket
struct ProfScope {
  int cls; hipStream_t st; hipEvent_t start{}, stop{}; bool live = false;
  ProfScope(int c, hipStream_t s, bool launches = true) : cls(c), st(s) {
    if (!g_prof_on || !launches) return;
    if (prof_event(&start) != DOMINO_OK || prof_event(&stop) != DOMINO_OK) return;
    if (hipEventRecord(start, st) != hipSuccess) return;
    live = true;
  }
  ~ProfScope() {
    if (!live) return;
    (void)hipEventRecord(stop, st);
    g_prof_recs.push_back({cls, st, start, stop});
  }
};

// launches in flight at once in the layer call being enqueued (tile choice of its GEMMs); 1 outside
thread_local int g_concurrency = 1;
thread_local int g_beside = 0;           // 1: the call's row groups run side by side (see GemmArgs::beside)
struct ConcurrencyScope {
  ConcurrencyScope(int c, const Layout& L) { g_concurrency = c < 1 ? 1 : c; g_beside = L.groups > 1; }
  ~ConcurrencyScope() { g_concurrency = 1; g_beside = 0; }
};

inline hipStream_t as_stream(void* s) { return static_cast<hipStream_t>(s); }
inline const char* at(const void* base, size_t off) { return static_cast<const char*>(base) + off; }
inline char* at(void* base, size_t off) { return static_cast<char*>(base) + off; }

GemmArgs gemm_args(const void* A, long lda, const void* B, long ldb, void* C, long ldc, int M, int N, int K) {
  GemmArgs a{};
  a.A = A; a.B = B; a.C = C; a.lda = lda; a.ldb = ldb; a.ldc = ldc; a.M = M; a.N = N; a.K = K;
  a.gelu_tanh = 1;
  a.concurrency = g_concurrency;
  a.beside = g_beside;
  return a;
}

// edge: work submitted later to `to` waits for everything submitted so far to `from`
int edge(hipStream_t from, hipStream_t to) {
  if (from == to) return DOMINO_OK;
  hipEvent_t ev;
  int rc = next_sync_event(&ev);
  if (rc != DOMINO_OK) return rc;
  HIP_TRY(hipEventRecord(ev, from), "hipEventRecord");
  HIP_TRY(hipStreamWaitEvent(to, ev, 0), "hipStreamWaitEvent");
  return DOMINO_OK;
}

#define TRY(expr)                      \
  do {                                 \
    int rc_ = (expr);                  \
    if (rc_ != DOMINO_OK) return rc_;  \
  } while (0)
#define LAUNCH(expr, what) HIP_TRY((expr), what)

int check_streams(void* const* streams, int nstreams) {
  if (!streams) return fail(DOMINO_ERR_NULL_POINTER, "streams is NULL");
  if (nstreams < 1 || nstreams > 64) return fail(DOMINO_ERR_INVALID_ARG, "nstreams %d outside [1, 64]", nstreams);
  return DOMINO_OK;
}

int check_params(const Layout& L, const domino_params* P) {
  if (!P) return fail(DOMINO_ERR_NULL_POINTER, "params is NULL");
  if (!P->norm1_g || !P->norm2_g || !P->w_qkv || !P->w_o || !P->w_up || !P->w_down)
    return fail(DOMINO_ERR_NULL_POINTER, "a weight matrix or norm gain pointer is NULL");
  if (L.llama) {
    if (P->norm1_b || P->norm2_b || P->b_qkv || P->b_o || P->b_up || P->b_down)
      return fail(DOMINO_ERR_INVALID_ARG, "the Llama architecture has no shifts or biases: those pointers must be NULL");
  } else if (!P->norm1_b || !P->norm2_b || !P->b_qkv || !P->b_o || !P->b_up || !P->b_down) {
    return fail(DOMINO_ERR_NULL_POINTER, "a GPT bias or norm shift pointer is NULL");
  }
  return DOMINO_OK;
}


// The QKV product applies the rotary embedding in its epilogue when a head's partner columns (i, i + d/2) can meet in
// one lane there: heads of 64 or 128 columns.  Other head sizes (80) take a separate in-place pass over q and k.
inline bool rope_fused(const Layout& L) { return L.llama && (L.d == 64 || L.d == 128); }

// ---------------------------------------------------------------------------------- the piece schedule
// One block's buffers as the forward / the backward sees them (all device pointers, caller-owned).
struct FwdLayer {
  const domino_params* P;
  const void *x, *attn_others, *mlp_others;
  void *attn_partial, *mlp_partial, *y, *saved;
};
struct BwdLayer {
  const domino_params* P;
  const domino_grads* G;
  const void *saved, *x, *dy, *dln2_others, *dln1_others;
  void *dln2_partial, *dln1_partial, *dx;
  float* red;        // this block's partial column sums: red_floats floats
  int accumulate;
};

// Which stream of the pool carries what (Sec. 4.3.1: a fixed pool, picked by index): row group g runs on streams[g], the
// backward's weight gradients on a stream of their own behind the groups' when the pool has one, where they fill the
// compute units that the chain of input gradients, attention and norms leaves idle (Sec. 4.1.2 runs a weight gradient
// beside the all-reduce of its input gradient).  Not under graph capture: instantiating a graph in which one stream
// waits for events of two others has crashed inside the runtime, so a captured call keeps to the groups' streams.
struct StreamPlan {
  void* const* streams;
  int ns, lanes;
  bool side;
  StreamPlan(void* const* s, int n, const Layout& L, int bwd_parts)
      : streams(s), ns(n), lanes(L.groups < n ? L.groups : n),
        side((bwd_parts & (DOMINO_BWD_MLP | DOMINO_BWD_ATTN)) && L.beside && !g_capturing && n > lanes) {}
  hipStream_t lane(int g) const { return as_stream(streams[g % lanes]); }
  hipStream_t side_stream() const { return as_stream(streams[lanes]); }
  int used() const { return lanes + (side ? 1 : 0); }
};

// fork: one event on streams[0]; every other stream that the call uses waits for it
int fork_streams(const StreamPlan& S, int n) {
  if (n < 2) return DOMINO_OK;
  hipEvent_t fork;
  TRY(next_sync_event(&fork));
  HIP_TRY(hipEventRecord(fork, as_stream(S.streams[0])), "hipEventRecord");
  for (int k = 1; k < n; ++k) HIP_TRY(hipStreamWaitEvent(as_stream(S.streams[k]), fork, 0), "hipStreamWaitEvent");
  return DOMINO_OK;
}
int join_streams(const StreamPlan& S, int n) {
  for (int k = 1; k < n; ++k) TRY(edge(as_stream(S.streams[k]), as_stream(S.streams[0])));
  return DOMINO_OK;
}

int check_fwd_layer(const Layout& L, const FwdLayer& B, int parts = DOMINO_FWD_ALL) {
  TRY(check_params(L, B.P));
  if (parts <= 0 || (parts & ~DOMINO_FWD_ALL)) return fail(DOMINO_ERR_INVALID_ARG, "forward parts %d outside [1, %d]", parts, (int)DOMINO_FWD_ALL);
  if (!B.x || !B.attn_partial || !B.saved) return fail(DOMINO_ERR_NULL_POINTER, "x, attn_partial or saved is NULL");
  if ((parts & DOMINO_FWD_MLP) && !B.mlp_partial) return fail(DOMINO_ERR_NULL_POINTER, "mlp_partial is NULL");
  return DOMINO_OK;
}

int check_bwd_layer(const Layout& L, const BwdLayer& B, int parts = DOMINO_BWD_ALL) {
  TRY(check_params(L, B.P));
  const domino_grads* G = B.G;
  if (parts <= 0 || (parts & ~DOMINO_BWD_ALL)) return fail(DOMINO_ERR_INVALID_ARG, "backward parts %d outside [1, %d]", parts, (int)DOMINO_BWD_ALL);
  if (!B.saved || !G) return fail(DOMINO_ERR_NULL_POINTER, "saved or grads is NULL");
  if ((parts & (DOMINO_BWD_MLP | DOMINO_BWD_ATTN)) && (!B.dy || !B.dln2_partial))
    return fail(DOMINO_ERR_NULL_POINTER, "dy or dln2_partial is NULL");
  if ((parts & (DOMINO_BWD_ATTN | DOMINO_BWD_NORM1)) && !B.dln1_partial) return fail(DOMINO_ERR_NULL_POINTER, "dln1_partial is NULL");
  if ((parts & DOMINO_BWD_NORM1) && (!B.x || !B.dx)) return fail(DOMINO_ERR_NULL_POINTER, "x or dx is NULL");
  if (!G->norm1_g || !G->norm2_g || !G->w_qkv || !G->w_o || !G->w_up || !G->w_down)
    return fail(DOMINO_ERR_NULL_POINTER, "a weight or norm-gain gradient pointer is NULL");
  if (!L.llama && (!G->norm1_b || !G->norm2_b || !G->b_qkv || !G->b_o || !G->b_up || !G->b_down))
    return fail(DOMINO_ERR_NULL_POINTER, "a GPT bias or norm-shift gradient pointer is NULL");
  if ((parts & DOMINO_BWD_MLP) && (parts & DOMINO_BWD_NORM1)) {      // the down-projection's weight gradient may read dy after dx is written
    const size_t bytes = (size_t)L.M * L.h * 2;
    const char *a = static_cast<const char*>(B.dy), *b = static_cast<const char*>(B.dx);
    if (a < b + bytes && b < a + bytes) return fail(DOMINO_ERR_INVALID_ARG, "dx overlaps dy");
  }
  return DOMINO_OK;
}

// The token rows that group g's launches cover.
struct Rows {
  size_t r0, rh;         // first row; byte offset of its hidden-wide bf16 row
  int n, batch, slice;   // rows, batch elements, first slice
};
Rows rows_of(const Layout& L, int g) {
  const int i0 = L.first_slice(g), i1 = L.first_slice(g + 1);
  const size_t r0 = (size_t)i0 * L.Ms;
  return {r0, r0 * L.h * 2, (i1 - i0) * L.Ms, (i1 - i0) * (L.b / L.p), i0};
}

// Forward of one block (Sec. 3.2, Eq. 3): each step of the block for one row group after the other, every group on its
// own stream.  The column pieces of each of the two row-cut products (Sec. 3.3, Eq. 4), written in place into the
// full-width buffers, are one launch: a piece is a unit of reduction, and inside a call none is handed out.  (With two groups the
// out-projection's once were a launch each, 26 us of which a third filled and drained the chip: 13B 2062 us, 2045 in one, 30B
// forward 1266 and 1256, Llama-2 13B 4181 and 4170, Llama-2 7B with 16 x 1024 tokens level.)
// `norm1_done`: the block's Norm1 has already been written (by the block below, see `next`).
// `next`: the block above in a stack; its Norm1 is then taken in the same pass that forms this block's output.
int enqueue_fwd_block(const Layout& L, const domino_cfg* cfg, const StreamPlan& S, const FwdLayer& B,
                      int parts = DOMINO_FWD_ALL, bool norm1_done = false, const FwdLayer* next = nullptr) {
  const domino_params* P = B.P;
  const bool rms = L.llama;
  void* saved = B.saved;
  auto rowf = [&](size_t off, const Rows& R) { return reinterpret_cast<float*>(at(saved, off)) + R.r0; };
  auto ln1 = [&](const Rows& R) { return at(saved, L.ln1 + R.rh); };
  auto qkv = [&](const Rows& R) { return at(saved, L.qkv + R.r0 * 3 * L.hl * 2); };
  auto ctx = [&](const Rows& R) { return at(saved, L.ctx + R.r0 * L.hl * 2); };
  auto x1 = [&](const Rows& R) { return at(saved, L.x1 + R.rh); };
  auto ln2 = [&](const Rows& R) { return at(saved, L.ln2 + R.rh); };
  auto act = [&](const Rows& R) { return at(saved, L.act + R.r0 * L.fl * 2); };
  auto each_group = [&](auto step) -> int {
    for (int g = 0; g < L.groups; ++g) TRY(step(rows_of(L, g), S.lane(g)));
    return DOMINO_OK;
  };

  if (parts & DOMINO_FWD_ATTN) {
    if (!norm1_done)
      TRY(each_group([&](const Rows& R, hipStream_t st) -> int {  // F1: Norm1
        ProfScope ps(PC_NORM_FWD, st);
        NormFwdArgs a{};
        a.x = at(B.x, R.rh); a.gamma = P->norm1_g; a.beta = P->norm1_b; a.y = ln1(R);
        a.mean = rms ? nullptr : rowf(L.mean1, R); a.rstd = rowf(L.rstd1, R);
        a.rows = R.n; a.h = L.h; a.rms = rms; a.eps = cfg->norm_eps;
        LAUNCH(norm_fwd_launch(a, st), "norm1 forward");
        return DOMINO_OK;
      }));
    TRY(each_group([&](const Rows& R, hipStream_t st) -> int {  // F2: X * A (attention), column-parallel, never column-sliced
      ProfScope ps(PC_GEMM_QKV, st);
      GemmArgs a = gemm_args(ln1(R), L.h, P->w_qkv, 3 * L.hl, qkv(R), 3 * L.hl, R.n, 3 * L.hl, L.h);
      a.bias = P->b_qkv;
      if (rope_fused(L)) {     // q and k leave the product already rotated (the rotary embedding of Sec. 5.4)
        a.rope_d = L.d; a.rope_seq = L.s; a.rope_cols = 2 * L.hl; a.rope_log2_base = log2f(cfg->rope_base);
        LAUNCH(gemm_launch(GEMM_NN, EPI_ROPE, a, -1, st), "qkv product");
      } else {
        LAUNCH(gemm_launch(GEMM_NN, EPI_STORE, a, -1, st), "qkv product");
      }
      return DOMINO_OK;
    }));
    if (L.llama && !rope_fused(L))
      TRY(each_group([&](const Rows& R, hipStream_t st) -> int {
        ProfScope ps(PC_ROPE, st);
        LAUNCH(rope_launch(qkv(R), 3 * L.hl, R.n, L.s, 0, 2, L.nl, L.d, cfg->rope_base, 0, st), "rotary embedding");
        return DOMINO_OK;
      }));
    TRY(each_group([&](const Rows& R, hipStream_t st) -> int {  // F3
      ProfScope ps(PC_ATTN_FWD, st);
      AttnArgs a{};
      a.qkv = qkv(R); a.ld = 3 * L.hl; a.ctx = ctx(R); a.ld_ctx = L.hl;
      a.lse = reinterpret_cast<float*>(at(saved, L.lse)) + R.r0 * L.nl;
      a.batch = R.batch; a.seq = L.s; a.heads = L.nl; a.head_dim = L.d; a.scale = 1.0f / sqrtf((float)L.d);
      LAUNCH(attention_fwd_launch(a, st), "attention forward");
      return DOMINO_OK;
    }));
    TRY(each_group([&](const Rows& R, hipStream_t st) -> int {  // F4: (XA) * B_j, all column pieces
      ProfScope ps(PC_GEMM_OUT, st);
      GemmArgs a = gemm_args(ctx(R), L.hl, P->w_o, L.h, at(B.attn_partial, R.rh), L.h, R.n, L.h, L.hl);
      LAUNCH(gemm_launch(GEMM_NN, EPI_STORE, a, -1, st), "out-projection");
      return DOMINO_OK;
    }));                                                    // column synchronisation before Norm2: stream order
  }
  if (!(parts & DOMINO_FWD_MLP)) return DOMINO_OK;
  TRY(each_group([&](const Rows& R, hipStream_t st) -> int {  // F5: residual + reduced attention output + Norm2
    ProfScope ps(PC_NORM_FWD, st);
    NormFwdArgs a{};
    a.x = at(B.x, R.rh); a.add1 = at(B.attn_partial, R.rh); a.add2 = B.attn_others ? at(B.attn_others, R.rh) : nullptr; a.vec = P->b_o;
    a.gamma = P->norm2_g; a.beta = P->norm2_b; a.xsum = x1(R); a.y = ln2(R);
    a.mean = rms ? nullptr : rowf(L.mean2, R); a.rstd = rowf(L.rstd2, R);
    a.rows = R.n; a.h = L.h; a.rms = rms; a.eps = cfg->norm_eps;
    LAUNCH(norm_fwd_launch(a, st), "norm2 forward");
    return DOMINO_OK;
  }));
  TRY(each_group([&](const Rows& R, hipStream_t st) -> int {  // F6: X * A (MLP) with the activation fused
    ProfScope ps(PC_GEMM_UP, st);
    GemmArgs a = gemm_args(ln2(R), L.h, P->w_up, L.upc, act(R), L.fl, R.n, L.fl, L.h);
    a.aux = at(saved, L.pre + R.r0 * L.upc * 2); a.ldaux = L.upc; a.gelu_tanh = cfg->gelu_tanh;
    if (L.llama) { a.n_split = L.fl; LAUNCH(gemm_launch(GEMM_NN, EPI_SWIGLU, a, -1, st), "mlp-up product"); }
    else { a.bias = P->b_up; LAUNCH(gemm_launch(GEMM_NN, EPI_BIAS_GELU, a, -1, st), "mlp-up product"); }
    return DOMINO_OK;
  }));
  // F8, the block output, in the product's epilogue where one row group is the chain and gemm_forms_output says so; with two
  // groups a pass, which runs beside the other group's product.  (Forward, us, pass and epilogue: 13B with 8192 tokens 721
  // and 738, Llama-2 7B with 16384 952 and 941, with 8 x 1024 532 and 535, 30B 1215 and 1208, Llama-2 13B 1387 and 1373;
  // their forward + backward is level to 1 %.)
  const bool y_in_product = B.y && !next && L.groups == 1 && gemm_forms_output(L.M, L.h, L.fl);
  TRY(each_group([&](const Rows& R, hipStream_t st) -> int {  // F7
    ProfScope ps(PC_GEMM_DOWN, st);
    GemmArgs a = gemm_args(act(R), L.fl, P->w_down, L.h, at(B.mlp_partial, R.rh), L.h, R.n, L.h, L.fl);
    if (y_in_product) {
      a.aux = x1(R); a.ldaux = L.h; a.add2 = B.mlp_others ? at(B.mlp_others, R.rh) : nullptr; a.bias = P->b_down; a.out2 = at(B.y, R.rh);
      LAUNCH(gemm_launch(GEMM_NN, EPI_RESID, a, -1, st), "mlp-down product and block output");
    } else {
      LAUNCH(gemm_launch(GEMM_NN, EPI_STORE, a, -1, st), "mlp-down product");
    }
    return DOMINO_OK;
  }));
  return each_group([&](const Rows& R, hipStream_t st) -> int {
    const void* others = B.mlp_others ? at(B.mlp_others, R.rh) : nullptr;
    if (next) {  // F8 of this block and F1 of the next in one pass over the rows: y is written and normalised at once
      ProfScope ps(PC_NORM_FWD, st);
      NormFwdArgs a{};
      a.x = x1(R); a.add1 = at(B.mlp_partial, R.rh); a.add2 = others; a.vec = P->b_down;
      a.gamma = next->P->norm1_g; a.beta = next->P->norm1_b; a.xsum = at(B.y, R.rh); a.y = at(next->saved, L.ln1 + R.rh);
      a.mean = rms ? nullptr : reinterpret_cast<float*>(at(next->saved, L.mean1)) + R.r0;
      a.rstd = reinterpret_cast<float*>(at(next->saved, L.rstd1)) + R.r0;
      a.rows = R.n; a.h = L.h; a.rms = rms; a.eps = cfg->norm_eps;
      LAUNCH(norm_fwd_launch(a, st), "block output + next norm1");
    } else if (B.y && !y_in_product) {
      ProfScope ps(PC_RESID_OUT, st);
      LAUNCH(residual_out_launch(x1(R), at(B.mlp_partial, R.rh), others, P->b_down, at(B.y, R.rh), (long)R.n * L.h, L.h, st), "block output");
    }
    return DOMINO_OK;
  });
}

// The gradients of a block's intermediate activations that its weight gradients read (whole tensors, all row slices).
struct GradBufs { char *d_pre, *dx1, *dqkv; };
GradBufs grad_bufs(const Layout& L, void* ws) { return {at(ws, L.d_pre), at(ws, L.dx1), at(ws, L.dqkv)}; }

// The weight gradients are not formed slice by slice: every slice after the first would read and rewrite the whole fp32
// gradient (for the 13B shard 0.94 GB of 9.4 GB per step at p = 4) in launches a p-th as deep.  With more than two slices
// a product is handed over once, over all rows; with one or two slice by slice and joined there (GemmArgs::join), to the
// same end.  cfg->wgrad_per_slice keeps the slice-by-slice launches of Sec. 4.1.2 for any p.
inline bool merged_wgrads(const Layout& L) { return L.merged; }

enum { WG_DOWN = 0, WG_UP, WG_OUT, WG_QKV, NWGRADS };

// the weight gradients of the n matrices in `which` and the column sums behind the biases of the same
// products, on `st`: one launch for all of them (`parts`: memory for the sums of L.wsplits contraction ranges, or NULL
// for one range); with cfg->wgrad_per_slice one per matrix and slice, in slice order, behind one per column sum.  `tail`: a Norm1 backward is held back
// for that one launch (HeldTail)
int weight_gradients(const Layout& L, const GradBufs& gb, const BwdLayer& B, const int* which, int n, hipStream_t st, float* parts, bool tail) {
  const char* sv = static_cast<const char*>(B.saved);
  const domino_grads* G = B.G;
  struct { int cls; const void* A; long lda; const void* Bm; long ldb; float* C; int M, N; int bias; } const tab[NWGRADS] = {
    {PC_WGRAD_DOWN, sv + L.act, L.fl, B.dy, L.h, G->w_down, L.fl, L.h, -1},
    {PC_WGRAD_UP, sv + L.ln2, L.h, gb.d_pre, L.upc, G->w_up, L.h, L.upc, AREA_BUP},
    {PC_WGRAD_OUT, sv + L.ctx, L.hl, gb.dx1, L.h, G->w_o, L.hl, L.h, -1},
    {PC_WGRAD_QKV, sv + L.ln1, L.h, gb.dqkv, 3 * L.hl, G->w_qkv, L.h, 3 * L.hl, AREA_BQKV}};
  struct Close { ~Close() { t_tail.open = false; } } close;      // nothing stays held back, whatever fails
  bool sums = false;
  for (int m = 0; m < n; ++m) sums |= !L.llama && tab[which[m]].bias >= 0;
  // with one row group the column sums are further workgroups of the weight gradients' launch (see gemm_tail_kernel of gemm.hip; with
  // two, where the chip is full, a 13B block's step is 0.5 % faster with launches of their own, 2029 and 2038 us)
  const bool held = tail || (sums && !L.per_slice && L.groups == 1);
  static_assert(COLSUM_MAX_HELD >= 2, "one group has a column sum for QKV and one for MLP-up, and both are held");
  if (held && !tail) t_tail = HeldTail{NormBwdArgs{}, {}, 0, st, true};
  for (int m = 0; m < n; ++m) {
    const auto& w = tab[which[m]];
    if (!L.llama && w.bias >= 0)
      for (int g = 0; g < L.groups; ++g) {
        const Rows R = rows_of(L, g);
        ProfScope ps(PC_COLSUM, st, !held);
        LAUNCH(colsum_partial_launch(at(w.Bm, R.r0 * w.ldb * 2), w.ldb, R.n, w.N, B.red + L.area(w.bias, g), st), "bias gradient");
      }
  }
  const int slices = merged_wgrads(L) ? 1 : L.p, K = L.M / slices;
  for (int m = 0; m < n; ++m) {
    const auto& w = tab[which[m]];
    for (int i = 0; i < slices; ++i) {
      const bool join = !L.per_slice && (m < n - 1 || i < slices - 1);
      ProfScope ps(n > 1 && !L.per_slice ? (int)PC_WGRAD_JOINED : w.cls, st, !join);
      const size_t r0 = (size_t)i * K;
      GemmArgs a = gemm_args(at(w.A, r0 * w.lda * 2), w.lda, at(w.Bm, r0 * w.ldb * 2), w.ldb, w.C, w.N, w.M, w.N, K);
      a.beta = (i > 0 || B.accumulate) ? 1 : 0;
      a.beside = L.beside;
      if (parts) { a.splits = L.wsplits; a.split_ws = parts; }
      a.join = join ? 1 : 0;
      a.tail = held ? 1 : 0;
      LAUNCH(gemm_launch(GEMM_TN, EPI_ACC_F32, a, -1, st), "weight gradient");
    }
  }
  return DOMINO_OK;
}

// The vector gradients (norm gains and shifts, biases) from the partial rows that the slices' norm backwards and the
// groups' column sums left: summed in index order, all slices in one launch (with cfg->wgrad_per_slice one per slice; the
// groups' column sums then belong to the first).  Those of the MLP half are complete behind the Norm2 backward, the
// others behind Norm1's.  All of them belong to the call that runs DOMINO_BWD_NORM1: only where that call holds the Norm2
// backward too may it reduce the MLP half's early.  The calls of one backward need not agree on their streams (another
// pool, one captured and the next not), so what an earlier part reduced could not be told from here.
enum { VEC_MLP = 1, VEC_ATTN = 2, VEC_ALL = 3 };
int vector_gradients(const Layout& L, const BwdLayer& B, int which, hipStream_t st) {
  const domino_grads* G = B.G;
  const int launches = merged_wgrads(L) ? 1 : L.p, slices = L.p / launches;
  for (int i = 0; i < launches; ++i) {
    const bool join = !L.per_slice && i < launches - 1;
    ProfScope ps(PC_COLSUM, st, !join);
    struct { int k; float* out; int set; } const vec[NAREAS] = {
      {AREA_G1, G->norm1_g, VEC_ATTN}, {AREA_B1, G->norm1_b, VEC_ATTN}, {AREA_G2, G->norm2_g, VEC_MLP}, {AREA_B2, G->norm2_b, VEC_MLP},
      {AREA_BQKV, G->b_qkv, VEC_ATTN}, {AREA_BO, G->b_o, VEC_MLP}, {AREA_BUP, G->b_up, VEC_MLP}, {AREA_BDOWN, G->b_down, VEC_MLP}};
    ColsumJobs jobs{};
    int njobs = 0;
    for (auto& v : vec) {
      if (!v.out || !(v.set & which)) continue;
      if (L.llama && v.k != AREA_G1 && v.k != AREA_G2) continue;
      const bool by_group = v.k == AREA_BQKV || v.k == AREA_BUP;
      if (by_group && i > 0) continue;
      jobs.job[njobs++] = {B.red + L.area(v.k, by_group ? 0 : i * slices), v.out, L.area_rows[v.k], L.area_n[v.k], (long)L.area_n[v.k],
                           by_group ? L.groups : slices, (long)L.area_rows[v.k] * L.area_n[v.k]};
    }
    jobs.join = join ? 1 : 0;
    LAUNCH(colsum_finish_jobs_launch(jobs, njobs, (i > 0 || B.accumulate) ? 1 : 0, st), "vector gradient reduction");
  }
  return DOMINO_OK;
}

// Whether the Norm1 backward and the bias gradients go into the weight gradients' launch where one stream carries them all: two
// or three launches fewer, which pays the more the smaller the block is (figures at gemm_tail_kernel of gemm.hip).  The Norm1
// backward apart and joined at the line, us: 4096 tokens of a 2048-wide block 348 and 342, 8192 of a 1024-wide one 300.5 and
// 302.8.  Beyond it the two go on like that (2048-wide, 6144 tokens 486 and 473, 8000 559 and 548; 1024-wide, 12288 tokens 435 and 438; 1536-wide,
// 5120 422 and 426, 10240 675 and 673).
inline bool tail_joins(const Layout& L) {
  return L.groups == 1 && !L.per_slice && L.wsplits == 1 && L.h <= HeldTail::MAX_H && (long)L.M * L.h <= 1L << 23;
}

// What the blocks of a stack hand on to each other: events behind the weight gradients of a block and the stream each ran
// on (the tensors they read are written again two blocks later), and behind its Norm1 backward, per group (it writes the
// dy of the block below).
struct BlockEvents {
  hipEvent_t wgrad[NWGRADS] = {};
  hipStream_t on[NWGRADS] = {};
  std::vector<hipEvent_t> dx;
};

int record(hipEvent_t* ev, hipStream_t st) {
  TRY(next_sync_event(ev));
  HIP_TRY(hipEventRecord(*ev, st), "hipEventRecord");
  return DOMINO_OK;
}
int wait(hipStream_t st, hipEvent_t ev) {
  if (ev) HIP_TRY(hipStreamWaitEvent(st, ev, 0), "hipStreamWaitEvent");
  return DOMINO_OK;
}

// Where the weight gradients run beside the chain, or the call is the Norm1 part alone, the streams meet on streams[0] before the last
// reduction of the vector gradients and not behind it: an edge between streams is 10 to 14 us in which nothing else runs, and on
// the side stream the reduction stood between two of them (forward + backward, us, both with the events as next_sync_event makes them:
// 13B with 2048 tokens 661 and 650, Llama-2 7B 1560 and 1538, the 13B block in parts 2170 and 2149).
inline bool reduces_joined(const StreamPlan& S, int parts) {
  return (parts & DOMINO_BWD_NORM1) && (S.side || !(parts & (DOMINO_BWD_MLP | DOMINO_BWD_ATTN)));
}

// Backward of one block: each step of the chain of input gradients for one row group after the other, every group on
// its own stream; each input gradient is enqueued before the weight gradient of the same product (Sec. 4.1.2).  With a
// side stream the weight and vector gradients run there, each behind an event of every group; without one they follow
// on the groups' streams: one group forms them where their operands are complete, several first meet on streams[0] and
// part again (the same join and fork that end one call and begin the next) and take the matrices in turn.
// `last`: no block follows in the call.  In a stack: `own` receives this block's events, `above` are those of the block above, `two_above` of the block that
// used the same set of gradient tensors (NULL outside a stack or where there is no such block); `turn` deals the matrices
// to the streams differently from block to block.
int enqueue_bwd_block(const Layout& L, const domino_cfg* cfg, const StreamPlan& S, void* ws, const GradBufs& gb, const BwdLayer& B,
                      int parts, bool last, int turn = 0, BlockEvents* own = nullptr, const BlockEvents* above = nullptr,
                      const BlockEvents* two_above = nullptr) {
  const domino_params* P = B.P;
  const void* saved = B.saved;
  const bool rms = L.llama;
  auto rowf = [&](size_t off, const Rows& R) { return reinterpret_cast<const float*>(at(saved, off)) + R.r0; };
  auto d_pre = [&](const Rows& R) { return gb.d_pre + R.r0 * L.upc * 2; };
  auto dx1 = [&](const Rows& R) { return gb.dx1 + R.rh; };
  auto dqkv = [&](const Rows& R) { return gb.dqkv + R.r0 * 3 * L.hl * 2; };
  auto dctx = [&](const Rows& R) { return at(ws, L.dctx + R.r0 * L.hl * 2); };
  auto each_group = [&](auto step) -> int {
    for (int g = 0; g < L.groups; ++g) TRY(step(rows_of(L, g), S.lane(g)));
    return DOMINO_OK;
  };
  // an event on every stream that carries groups: `to` then waits for what the groups have enqueued so far
  auto behind_groups = [&](hipStream_t to, std::vector<hipEvent_t>* keep = nullptr) -> int {
    for (int k = 0; k < S.lanes; ++k) {
      hipEvent_t ev;
      TRY(record(&ev, as_stream(S.streams[k])));
      if (keep) keep->push_back(ev);
      if (to != as_stream(S.streams[k])) TRY(wait(to, ev));
    }
    return DOMINO_OK;
  };
  const bool in_place = !S.side && S.lanes == 1;
  // several contraction ranges where the launch follows the chain on its one stream: nothing else then uses their sums' memory
  float* const parts_ws = in_place && L.wsplits > 1 ? reinterpret_cast<float*>(at(ws, L.wpart)) : nullptr;
  auto form = [&](std::initializer_list<int> which, hipStream_t st, bool tail = false) -> int {
    TRY(weight_gradients(L, gb, B, which.begin(), (int)which.size(), st, parts_ws, tail));
    if (own) {
      hipEvent_t ev;
      TRY(record(&ev, st));
      for (int m : which) { own->on[m] = st; own->wgrad[m] = ev; }
    }
    return DOMINO_OK;
  };
  hipStream_t side = S.side ? S.side_stream() : nullptr;
  const bool mlp_vectors_early = S.side && (parts & DOMINO_BWD_ATTN) && (parts & DOMINO_BWD_NORM1);

  // the set of gradient tensors that this block writes was read by the weight gradients of the block two above, enqueued
  // a whole block ago: these waits order without stalling (on the side stream the last of them is behind the others)
  if (two_above)
    for (int k = 0; k < S.lanes; ++k)
      for (int m = S.side ? WG_QKV : WG_UP; m < NWGRADS; ++m)
        if (two_above->on[m] != as_stream(S.streams[k])) TRY(wait(as_stream(S.streams[k]), two_above->wgrad[m]));

  auto norm_bwd = [&](const Rows& R, hipStream_t st, const void* ga, const void* gb2, const void* xin, const void* gamma, size_t mean,
                      size_t rstd, const void* dres, void* out, int kg, int kb, int kres, int kdx, bool join = false) -> int {
    ProfScope ps(PC_NORM_BWD, st, !join);
    NormBwdArgs a{};
    a.ga = ga; a.gb = gb2; a.x = xin; a.gamma = gamma; a.mean = rowf(mean, R); a.rstd = rowf(rstd, R); a.dres = dres; a.dx = out;
    a.part_g = B.red + L.area(kg, R.slice); a.part_b = B.red + L.area(kb, R.slice); a.rows = R.n; a.h = L.h; a.rms = rms;
    a.slice_rows = L.Ms;
    a.slice_blocks = L.area_rows[kg];
    a.join = join ? 1 : 0;
    if (kres >= 0) { a.part_dres = B.red + L.area(kres, R.slice); a.part_dx = B.red + L.area(kdx, R.slice); }   // bias gradients of the two row-cut products
    LAUNCH(norm_bwd_launch(a, st), "norm backward");
    return DOMINO_OK;
  };

  auto norm1 = [&](bool join) -> int {
    // in a stack dx goes into the tensor that the block above took its dy from, and that block's down-projection weight
    // gradient, enqueued a whole block ago, reads all of it
    if (above && above->wgrad[WG_DOWN])
      for (int k = 0; k < S.lanes; ++k)
        if (above->on[WG_DOWN] != as_stream(S.streams[k])) TRY(wait(as_stream(S.streams[k]), above->wgrad[WG_DOWN]));
    return each_group([&](const Rows& R, hipStream_t st) -> int {
      return norm_bwd(R, st, at(B.dln1_partial, R.rh), B.dln1_others ? at(B.dln1_others, R.rh) : nullptr, at(B.x, R.rh), P->norm1_g,
                      L.mean1, L.rstd1, dx1(R), at(B.dx, R.rh), AREA_G1, AREA_B1, -1, -1, join);
    });
  };
  const bool joined_tail = in_place && (parts & DOMINO_BWD_ATTN) && (parts & DOMINO_BWD_NORM1) && tail_joins(L);

  if (parts & DOMINO_BWD_MLP) {
    if (S.side) {        // operands: the forward's, and dy, which in a stack the block above has just written
      if (above) for (hipEvent_t ev : above->dx) TRY(wait(side, ev));
      TRY(form({WG_DOWN}, side));                           // B2
    }
    TRY(each_group([&](const Rows& R, hipStream_t st) -> int {
      // B1 + B3: input gradient of the down-projection (all q column slices inside the K loop), activation backward fused
      ProfScope ps(PC_DGRAD_DOWN, st);
      GemmArgs a = gemm_args(at(B.dy, R.rh), L.h, P->w_down, L.h, d_pre(R), L.upc, R.n, L.fl, L.h);
      a.aux = const_cast<char*>(at(saved, L.pre + R.r0 * L.upc * 2)); a.ldaux = L.upc; a.gelu_tanh = cfg->gelu_tanh;
      if (L.llama) { a.n_split = L.fl; LAUNCH(gemm_launch(GEMM_NT, EPI_DSWIGLU, a, -1, st), "mlp-down input gradient"); }
      else LAUNCH(gemm_launch(GEMM_NT, EPI_DGELU, a, -1, st), "mlp-down input gradient");
      return DOMINO_OK;
    }));
    if (S.side) {
      TRY(behind_groups(side));
      TRY(form({WG_UP}, side));
    }
    TRY(each_group([&](const Rows& R, hipStream_t st) -> int {
      // B4: input gradient of MLP-up: the tensor the third all-reduce would sum
      ProfScope ps(PC_DGRAD_UP, st);
      GemmArgs a = gemm_args(d_pre(R), L.upc, P->w_up, L.upc, at(B.dln2_partial, R.rh), L.h, R.n, L.h, L.upc);
      LAUNCH(gemm_launch(GEMM_NT, EPI_STORE, a, -1, st), "mlp-up input gradient");
      return DOMINO_OK;
    }));
    if (in_place && !(parts & DOMINO_BWD_ATTN)) TRY(form({WG_DOWN, WG_UP}, S.lane(0)));
  }
  if (parts & DOMINO_BWD_ATTN) {
    TRY(each_group([&](const Rows& R, hipStream_t st) -> int {  // B5
      return norm_bwd(R, st, at(B.dln2_partial, R.rh), B.dln2_others ? at(B.dln2_others, R.rh) : nullptr, at(saved, L.x1 + R.rh),
                      P->norm2_g, L.mean2, L.rstd2, at(B.dy, R.rh), dx1(R), AREA_G2, AREA_B2, L.llama ? -1 : AREA_BDOWN, L.llama ? -1 : AREA_BO);
    }));
    if (S.side) {
      // one group: beside the attention backward, which leaves the matrix cores idle most of the time; two groups leave
      // little idle there, and the few tiles of the out-projection then share a launch with QKV's (2826 -> 2694 us for
      // 16384 tokens of Llama-2 7B; 13B equal; 2048 tokens of 13B in one group 701 -> 708)
      TRY(behind_groups(side));
      if (L.groups == 1) TRY(form({WG_OUT}, side));
      if (mlp_vectors_early) TRY(vector_gradients(L, B, VEC_MLP, side));
    }
    TRY(each_group([&](const Rows& R, hipStream_t st) -> int {  // B6
      ProfScope ps(PC_DGRAD_OUT, st);
      GemmArgs a = gemm_args(dx1(R), L.h, P->w_o, L.h, dctx(R), L.hl, R.n, L.hl, L.h);
      LAUNCH(gemm_launch(GEMM_NT, EPI_STORE, a, -1, st), "out-projection input gradient");
      return DOMINO_OK;
    }));
    TRY(each_group([&](const Rows& R, hipStream_t st) -> int {  // B7
      ProfScope ps(PC_ATTN_BWD, st);
      AttnArgs a{};
      a.qkv = at(saved, L.qkv + R.r0 * 3 * L.hl * 2); a.ld = 3 * L.hl;
      a.ctx = const_cast<char*>(at(saved, L.ctx + R.r0 * L.hl * 2)); a.ld_ctx = L.hl; a.dctx = dctx(R);
      a.lse = const_cast<float*>(reinterpret_cast<const float*>(at(saved, L.lse))) + R.r0 * L.nl;
      a.dot = reinterpret_cast<float*>(at(ws, L.dot)) + R.r0 * L.nl; a.dqkv = dqkv(R);
      a.batch = R.batch; a.seq = L.s; a.heads = L.nl; a.head_dim = L.d; a.scale = 1.0f / sqrtf((float)L.d);
      a.rope = L.llama ? 1 : 0; a.rope_log2_base = log2f(cfg->rope_base);   // dq, dk are turned back where they are stored
      LAUNCH(attention_bwd_launch(a, st), "attention backward");
      return DOMINO_OK;
    }));
    if (S.side) {
      TRY(behind_groups(side));
      if (L.groups == 1) TRY(form({WG_QKV}, side));
      else TRY(form({WG_OUT, WG_QKV}, side));
    }
    TRY(each_group([&](const Rows& R, hipStream_t st) -> int {
      // B8: input gradient of QKV: the tensor the fourth all-reduce would sum
      ProfScope ps(PC_DGRAD_QKV, st);
      GemmArgs a = gemm_args(dqkv(R), 3 * L.hl, P->w_qkv, 3 * L.hl, at(B.dln1_partial, R.rh), L.h, R.n, L.h, 3 * L.hl);
      LAUNCH(gemm_launch(GEMM_NT, EPI_STORE, a, -1, st), "qkv input gradient");
      return DOMINO_OK;
    }));
    if (in_place) {      // all of the call's weight gradients in one launch
      if (joined_tail) TRY(norm1(true));
      if (parts & DOMINO_BWD_MLP) TRY(form({WG_DOWN, WG_UP, WG_OUT, WG_QKV}, S.lane(0), joined_tail));
      else TRY(form({WG_OUT, WG_QKV}, S.lane(0), joined_tail));
    }
  }
  if ((parts & DOMINO_BWD_NORM1) && !joined_tail) TRY(norm1(false));
  if (last && reduces_joined(S, parts)) {
    TRY(join_streams(S, S.used()));
    TRY(vector_gradients(L, B, mlp_vectors_early ? VEC_ATTN : VEC_ALL, S.lane(0)));
  } else if (S.side) {
    if (parts & DOMINO_BWD_NORM1) {
      TRY(behind_groups(side, own ? &own->dx : nullptr));
      TRY(vector_gradients(L, B, mlp_vectors_early ? VEC_ATTN : VEC_ALL, side));
    }
  } else if (in_place) {
    if (parts & DOMINO_BWD_NORM1) TRY(vector_gradients(L, B, VEC_ALL, S.lane(0)));
  } else {
    TRY(join_streams(S, S.lanes));
    TRY(fork_streams(S, S.lanes));
    int slot = turn;
    const int order[NWGRADS] = {WG_DOWN, WG_UP, WG_QKV, WG_OUT};
    for (int which : order)
      if (parts & (which <= WG_UP ? DOMINO_BWD_MLP : DOMINO_BWD_ATTN)) TRY(form({which}, as_stream(S.streams[slot++ % S.lanes])));
    if (parts & DOMINO_BWD_NORM1) {
      // behind the column sums, which come with the matrices, on whichever stream they ran
      if (!L.llama && (parts & (DOMINO_BWD_MLP | DOMINO_BWD_ATTN))) {
        TRY(join_streams(S, S.lanes));
        TRY(fork_streams(S, S.lanes));
      }
      TRY(vector_gradients(L, B, VEC_ALL, as_stream(S.streams[slot % S.lanes])));
    }
  }
  return DOMINO_OK;
}

// workspace of a stack: one block's workspace, the partial-sum areas of the other blocks, two gradient tensors
// handed from block to block in turn (a block reads its dy from one and writes its dx into the other) and, where weight
// gradients run beside the chain, a second set of the tensors they read, so that the block below can run on meanwhile
struct StackLayout {
  size_t red_bytes, extra_red, dmid[2], d_pre2, dx1_2, dqkv2, total;
};
StackLayout stack_layout(const Layout& L, int nlayers) {
  StackLayout s{};
  const size_t Mz = (size_t)L.M;
  s.red_bytes = align_up(L.red_floats * 4);
  s.extra_red = L.ws_total;
  size_t o = s.extra_red + (size_t)(nlayers - 1) * s.red_bytes;
  auto take = [&](size_t bytes) { size_t at = o; o += align_up(bytes); return at; };
  s.dmid[0] = take(Mz * L.h * 2);
  s.dmid[1] = take(Mz * L.h * 2);
  if (nlayers > 1 && L.beside) {
    s.d_pre2 = take(Mz * L.upc * 2);
    s.dx1_2 = take(Mz * L.h * 2);
    s.dqkv2 = take(Mz * 3 * L.hl * 2);
  }
  s.total = o;
  return s;
}
constexpr int MAX_STACK_LAYERS = 1024;

}  // namespace

extern "C" {

const char* domino_last_error(void) { return g_err; }
const char* domino_last_warning(void) {
  std::lock_guard<std::mutex> lock(g_warn_mutex);
  return g_warn;
}
int domino_capture_supported(int nstreams, int p) {
  return (nstreams >= 1 && p >= 1 && capture_pool_ok(nstreams, p)) ? 1 : 0;
}
const char* domino_version(void) { return "domino-mi355x 0.1 (gfx950)"; }

int domino_validate_cfg(const domino_cfg* cfg) { return validate(cfg, nullptr); }

size_t domino_saved_bytes(const domino_cfg* cfg) {
  Layout L;
  return validate(cfg, &L) == DOMINO_OK ? L.saved_total : 0;
}
size_t domino_workspace_bytes(const domino_cfg* cfg) {
  Layout L;
  return validate(cfg, &L) == DOMINO_OK ? L.ws_total : 0;
}

int domino_saved_slot(const domino_cfg* cfg, const char* name, size_t* offset, size_t* bytes) {
  Layout L;
  TRY(validate(cfg, &L));
  if (!name || !offset || !bytes) return fail(DOMINO_ERR_NULL_POINTER, "name, offset or bytes is NULL");
  const size_t Mz = (size_t)L.M;
  struct { const char* n; size_t off, sz; } tab[] = {
    {"ln1", L.ln1, Mz * L.h * 2}, {"qkv", L.qkv, Mz * 3 * L.hl * 2}, {"ctx", L.ctx, Mz * L.hl * 2},
    {"lse", L.lse, (size_t)L.b * L.nl * L.s * 4}, {"x1", L.x1, Mz * L.h * 2}, {"ln2", L.ln2, Mz * L.h * 2},
    {"pre", L.pre, Mz * L.upc * 2}, {"act", L.act, Mz * L.fl * 2}, {"mean1", L.mean1, Mz * 4},
    {"rstd1", L.rstd1, Mz * 4}, {"mean2", L.mean2, Mz * 4}, {"rstd2", L.rstd2, Mz * 4}};
  for (auto& e : tab)
    if (!strcmp(e.n, name)) { *offset = e.off; *bytes = e.sz; return DOMINO_OK; }
  return fail(DOMINO_ERR_INVALID_ARG, "unknown saved tensor '%s'", name);
}

// ------------------------------------------------------------------------------------ forward
int domino_layer_fwd(const domino_cfg* cfg, const domino_params* P,
                     const void* x, const void* attn_others, const void* mlp_others,
                     void* attn_partial, void* mlp_partial, void* y,
                     void* saved, void* workspace, size_t workspace_bytes,
                     void* const* streams, int nstreams) {
  return domino_layer_fwd_parts(cfg, P, x, attn_others, mlp_others, attn_partial, mlp_partial, y, saved, workspace,
                                workspace_bytes, streams, nstreams, DOMINO_FWD_ALL);
}

int domino_layer_fwd_parts(const domino_cfg* cfg, const domino_params* P,
                           const void* x, const void* attn_others, const void* mlp_others,
                           void* attn_partial, void* mlp_partial, void* y,
                           void* saved, void* workspace, size_t workspace_bytes,
                           void* const* streams, int nstreams, int parts) {
  Layout L;
  TRY(validate(cfg, &L));
  const FwdLayer B{P, x, attn_others, mlp_others, attn_partial, mlp_partial, y, saved};
  TRY(check_fwd_layer(L, B, parts));
  TRY(check_streams(streams, nstreams));
  if (!workspace) return fail(DOMINO_ERR_NULL_POINTER, "workspace is NULL");
  if (workspace_bytes < L.ws_total) return fail(DOMINO_ERR_WORKSPACE_TOO_SMALL, "workspace holds %zu bytes, %zu needed", workspace_bytes, L.ws_total);
  std::lock_guard<std::mutex> lock(g_mutex);
  TRY(begin_call(streams, nstreams, L.p));
  const StreamPlan S(streams, nstreams, L, 0);
  note_hw_queues(S.used());
  ConcurrencyScope conc(S.used(), L);
  TRY(fork_streams(S, S.used()));
  TRY(enqueue_fwd_block(L, cfg, S, B, parts));
  TRY(join_streams(S, S.used()));
  return DOMINO_OK;
}

// ------------------------------------------------------------------------------------ backward
int domino_layer_bwd(const domino_cfg* cfg, const domino_params* P, const void* saved,
                     const void* x, const void* dy,
                     const void* dln2_others, const void* dln1_others,
                     void* dln2_partial, void* dln1_partial, void* dx,
                     const domino_grads* G, int accumulate,
                     void* workspace, size_t workspace_bytes,
                     void* const* streams, int nstreams) {
  return domino_layer_bwd_parts(cfg, P, saved, x, dy, dln2_others, dln1_others, dln2_partial, dln1_partial, dx, G,
                                accumulate, workspace, workspace_bytes, streams, nstreams, DOMINO_BWD_ALL);
}

int domino_layer_bwd_parts(const domino_cfg* cfg, const domino_params* P, const void* saved,
                           const void* x, const void* dy,
                           const void* dln2_others, const void* dln1_others,
                           void* dln2_partial, void* dln1_partial, void* dx,
                           const domino_grads* G, int accumulate,
                           void* workspace, size_t workspace_bytes,
                           void* const* streams, int nstreams, int parts) {
  Layout L;
  TRY(validate(cfg, &L));
  BwdLayer B{P, G, saved, x, dy, dln2_others, dln1_others, dln2_partial, dln1_partial, dx, nullptr, accumulate};
  TRY(check_bwd_layer(L, B, parts));
  TRY(check_streams(streams, nstreams));
  if (!workspace) return fail(DOMINO_ERR_NULL_POINTER, "workspace is NULL");
  if (workspace_bytes < L.ws_total) return fail(DOMINO_ERR_WORKSPACE_TOO_SMALL, "workspace holds %zu bytes, %zu needed", workspace_bytes, L.ws_total);
  std::lock_guard<std::mutex> lock(g_mutex);
  TRY(begin_call(streams, nstreams, L.p));
  B.red = reinterpret_cast<float*>(at(workspace, L.red));
  const StreamPlan S(streams, nstreams, L, parts);
  note_hw_queues(S.used());
  ConcurrencyScope conc(S.used(), L);
  TRY(fork_streams(S, S.used()));
  TRY(enqueue_bwd_block(L, cfg, S, workspace, grad_bufs(L, workspace), B, parts, true));
  if (!reduces_joined(S, parts)) TRY(join_streams(S, S.used()));
  return DOMINO_OK;
}

// ------------------------------------------------------------------------------------ stack of blocks
size_t domino_stack_workspace_bytes(const domino_cfg* cfg, int nlayers) {
  Layout L;
  if (validate(cfg, &L) != DOMINO_OK) return 0;
  if (nlayers < 1 || nlayers > MAX_STACK_LAYERS) { fail(DOMINO_ERR_INVALID_ARG, "nlayers %d outside [1, %d]", nlayers, MAX_STACK_LAYERS); return 0; }
  return stack_layout(L, nlayers).total;
}

int domino_stack_fwd(const domino_cfg* cfg, int nlayers, const domino_params* params, const void* x,
                     const domino_stack_fwd_io* io, void* workspace, size_t workspace_bytes,
                     void* const* streams, int nstreams) {
  Layout L;
  TRY(validate(cfg, &L));
  if (nlayers < 1 || nlayers > MAX_STACK_LAYERS) return fail(DOMINO_ERR_INVALID_ARG, "nlayers %d outside [1, %d]", nlayers, MAX_STACK_LAYERS);
  if (!params || !io) return fail(DOMINO_ERR_NULL_POINTER, "params or io is NULL");
  std::vector<FwdLayer> layers(nlayers);
  for (int l = 0; l < nlayers; ++l) {
    layers[l] = FwdLayer{&params[l], l == 0 ? x : io[l - 1].y, io[l].attn_others, io[l].mlp_others,
                         io[l].attn_partial, io[l].mlp_partial, io[l].y, io[l].saved};
    TRY(check_fwd_layer(L, layers[l]));
    if (!io[l].y) return fail(DOMINO_ERR_NULL_POINTER, "y of block %d is NULL: a stack needs every block's output", l);
  }
  TRY(check_streams(streams, nstreams));
  const size_t need = stack_layout(L, nlayers).total;
  if (!workspace) return fail(DOMINO_ERR_NULL_POINTER, "workspace is NULL");
  if (workspace_bytes < need) return fail(DOMINO_ERR_WORKSPACE_TOO_SMALL, "workspace holds %zu bytes, %zu needed", workspace_bytes, need);
  std::lock_guard<std::mutex> lock(g_mutex);
  TRY(begin_call(streams, nstreams, L.p));
  // a row slice of block l+1 needs only the same row slice of block l (Sec. 3.2): the groups run through the
  // whole stack on their own streams and meet only at the end
  const StreamPlan S(streams, nstreams, L, 0);
  note_hw_queues(S.used());
  ConcurrencyScope conc(S.used(), L);
  TRY(fork_streams(S, S.used()));
  for (int l = 0; l < nlayers; ++l)
    TRY(enqueue_fwd_block(L, cfg, S, layers[l], DOMINO_FWD_ALL, l > 0, l + 1 < nlayers ? &layers[l + 1] : nullptr));
  TRY(join_streams(S, S.used()));
  return DOMINO_OK;
}

int domino_stack_bwd(const domino_cfg* cfg, int nlayers, const domino_params* params, const void* dy,
                     const domino_stack_bwd_io* io, void* dx, const domino_grads* grads, int accumulate,
                     void* workspace, size_t workspace_bytes, void* const* streams, int nstreams) {
  Layout L;
  TRY(validate(cfg, &L));
  if (nlayers < 1 || nlayers > MAX_STACK_LAYERS) return fail(DOMINO_ERR_INVALID_ARG, "nlayers %d outside [1, %d]", nlayers, MAX_STACK_LAYERS);
  if (!params || !io || !grads) return fail(DOMINO_ERR_NULL_POINTER, "params, io or grads is NULL");
  if (!workspace) return fail(DOMINO_ERR_NULL_POINTER, "workspace is NULL");
  const StackLayout SL = stack_layout(L, nlayers);
  if (workspace_bytes < SL.total) return fail(DOMINO_ERR_WORKSPACE_TOO_SMALL, "workspace holds %zu bytes, %zu needed", workspace_bytes, SL.total);
  std::vector<BwdLayer> layers(nlayers);
  for (int l = 0; l < nlayers; ++l) {
    float* red = reinterpret_cast<float*>(l == 0 ? at(workspace, L.red) : at(workspace, SL.extra_red + (size_t)(l - 1) * SL.red_bytes));
    // the gradient handed down the stack lives in two tensors taken in turn: a slice's last kernel of block l writes
    // the rows that the same slice of block l-1, next on the same stream, reads
    const int turn = (nlayers - 1 - l) & 1;
    layers[l] = BwdLayer{&params[l], &grads[l], io[l].saved, io[l].x, l == nlayers - 1 ? dy : at(workspace, SL.dmid[turn ^ 1]),
                         io[l].dln2_others, io[l].dln1_others, io[l].dln2_partial, io[l].dln1_partial,
                         l == 0 ? dx : at(workspace, SL.dmid[turn]), red, accumulate};
    TRY(check_bwd_layer(L, layers[l]));
  }
  TRY(check_streams(streams, nstreams));
  std::lock_guard<std::mutex> lock(g_mutex);
  TRY(begin_call(streams, nstreams, L.p));
  const bool merged = merged_wgrads(L);
  // A graph captured from this call with merged weight gradients and more than one block crashed the runtime when
  // it was instantiated (the single-block call, whose capture is a chain of plain forks and joins, replays fine):
  // refused until the cause is known.
  if (g_capturing && merged && nlayers > 1)
    return fail(DOMINO_ERR_UNSUPPORTED, "streams[0] is being captured into a HIP graph: the backward of a stack of %d blocks with "
                "p = %d > 2 row slices cannot be captured; capture one domino_layer_bwd call per block instead", nlayers, L.p);
  const StreamPlan S(streams, nstreams, L, DOMINO_BWD_ALL);
  note_hw_queues(S.used());
  ConcurrencyScope conc(S.used(), L);
  TRY(fork_streams(S, S.used()));
  GradBufs gb[2] = {grad_bufs(L, workspace), grad_bufs(L, workspace)};
  if (nlayers > 1 && L.beside) gb[1] = GradBufs{at(workspace, SL.d_pre2), at(workspace, SL.dx1_2), at(workspace, SL.dqkv2)};
  // by set of gradient tensors: what the last block that used it left for the others to wait for
  BlockEvents ev[2];
  const bool several = S.used() > 1;       // one stream orders itself
  for (int l = nlayers - 1, k = 0; l >= 0; --l, ++k) {
    BlockEvents own;
    TRY(enqueue_bwd_block(L, cfg, S, workspace, gb[k & 1], layers[l], DOMINO_BWD_ALL, l == 0, k, several ? &own : nullptr,
                          several && k > 0 ? &ev[(k & 1) ^ 1] : nullptr, several && k > 1 ? &ev[k & 1] : nullptr));
    ev[k & 1] = own;
  }
  if (!reduces_joined(S, DOMINO_BWD_ALL)) TRY(join_streams(S, S.used()));
  return DOMINO_OK;
}

// ------------------------------------------------------------------------------------ single kernels
int domino_gemm(int layout, int epilogue, int tile,
                const void* A, int64_t lda, const void* B, int64_t ldb, void* C, int64_t ldc,
                int M, int N, int K, const void* bias, void* aux, int64_t ldaux,
                int n_split, int beta, int gelu_tanh, void* stream) {
  if (!A || !B || !C) return fail(DOMINO_ERR_NULL_POINTER, "A, B or C is NULL");
  if (M <= 0 || N <= 0 || K <= 0) return fail(DOMINO_ERR_INVALID_ARG, "M, N, K must be positive");
  if (M % 8 || N % 8 || K % 8 || lda % 8 || ldb % 8 || ldc % 4) return fail(DOMINO_ERR_UNSUPPORTED, "dimensions must be multiples of 8");
  if (tile < -1 || tile > 3) return fail(DOMINO_ERR_INVALID_ARG, "tile %d outside [-1, 3]", tile);
  const bool ok = (layout == DOMINO_GEMM_NN && (epilogue == DOMINO_EPI_STORE || epilogue == DOMINO_EPI_BIAS_GELU || epilogue == DOMINO_EPI_SWIGLU)) ||
                  (layout == DOMINO_GEMM_NT && (epilogue == DOMINO_EPI_STORE || epilogue == DOMINO_EPI_DGELU || epilogue == DOMINO_EPI_DSWIGLU)) ||
                  (layout == DOMINO_GEMM_TN && epilogue == DOMINO_EPI_ACC_F32);
  if (!ok) return fail(DOMINO_ERR_INVALID_ARG, "epilogue %d is not defined for layout %d", epilogue, layout);
  const bool needs_aux = epilogue == DOMINO_EPI_BIAS_GELU || epilogue == DOMINO_EPI_SWIGLU || epilogue == DOMINO_EPI_DGELU || epilogue == DOMINO_EPI_DSWIGLU;
  if (needs_aux && !aux) return fail(DOMINO_ERR_NULL_POINTER, "this epilogue needs aux");
  if (needs_aux && ldaux % 8) return fail(DOMINO_ERR_UNSUPPORTED, "ldaux must be a multiple of 8");
  if (epilogue == DOMINO_EPI_SWIGLU || epilogue == DOMINO_EPI_DSWIGLU) {
    if (n_split != N) return fail(DOMINO_ERR_INVALID_ARG, "SwiGLU epilogues need n_split == N");
    if (epilogue == DOMINO_EPI_SWIGLU && n_split % 32) return fail(DOMINO_ERR_UNSUPPORTED, "n_split must be a multiple of 32");
  }
  GemmArgs a = gemm_args(A, lda, B, ldb, C, ldc, M, N, K);
  a.bias = bias; a.aux = aux; a.ldaux = ldaux; a.n_split = n_split; a.beta = beta; a.gelu_tanh = gelu_tanh;
  const long wide_b = (layout == DOMINO_GEMM_NT) ? ((long)(N - 1) * ldb + K) : ((long)(K - 1) * ldb + (epilogue == DOMINO_EPI_SWIGLU ? 2L * N : N));
  const long wide_a = (layout == DOMINO_GEMM_TN) ? ((long)(K - 1) * lda + M) : ((long)(M - 1) * lda + K);
  if (wide_a * 2 >= TWO_GIB || wide_b * 2 >= TWO_GIB) return fail(DOMINO_ERR_UNSUPPORTED, "an operand would reach 2 GiB");
  HIP_TRY(gemm_launch(layout, epilogue, a, tile, as_stream(stream)), "gemm launch");
  return DOMINO_OK;
}

int domino_gemm_rope(int tile, const void* A, int64_t lda, const void* B, int64_t ldb, void* C, int64_t ldc,
                     int M, int N, int K, int seq, int head_dim, int rope_cols, float base, void* stream) {
  if (!A || !B || !C) return fail(DOMINO_ERR_NULL_POINTER, "A, B or C is NULL");
  if (M <= 0 || N <= 0 || K <= 0 || seq <= 0) return fail(DOMINO_ERR_INVALID_ARG, "M, N, K, seq must be positive");
  if (M % 8 || N % 8 || K % 8 || lda % 8 || ldb % 8 || ldc % 8) return fail(DOMINO_ERR_UNSUPPORTED, "dimensions must be multiples of 8");
  if (tile < -1 || tile > 3) return fail(DOMINO_ERR_INVALID_ARG, "tile %d outside [-1, 3]", tile);
  if (head_dim != 64 && head_dim != 128) return fail(DOMINO_ERR_UNSUPPORTED, "the rotary epilogue takes heads of 64 or 128 columns, not %d", head_dim);
  if (N % head_dim || rope_cols < 0 || rope_cols > N || rope_cols % head_dim)
    return fail(DOMINO_ERR_INVALID_ARG, "N and rope_cols must be multiples of head_dim, rope_cols <= N");
  if (!(base > 1.0f)) return fail(DOMINO_ERR_INVALID_ARG, "base must exceed 1");
  if (((long)(M - 1) * lda + K) * 2 >= TWO_GIB || ((long)(K - 1) * ldb + N) * 2 >= TWO_GIB) return fail(DOMINO_ERR_UNSUPPORTED, "an operand would reach 2 GiB");
  GemmArgs a = gemm_args(A, lda, B, ldb, C, ldc, M, N, K);
  a.rope_d = head_dim; a.rope_seq = seq; a.rope_cols = rope_cols; a.rope_log2_base = log2f(base);
  HIP_TRY(gemm_launch(GEMM_NN, EPI_ROPE, a, tile, as_stream(stream)), "gemm launch");
  return DOMINO_OK;
}

int domino_norm_fwd(const void* x, const void* add1, const void* add2, const void* vec,
                    const void* gamma, const void* beta, void* xsum, void* y, float* mean, float* rstd,
                    int rows, int h, int rms, float eps, void* stream) {
  if (!x || !gamma || !y || !rstd) return fail(DOMINO_ERR_NULL_POINTER, "x, gamma, y or rstd is NULL");
  if (rows <= 0 || h <= 0) return fail(DOMINO_ERR_INVALID_ARG, "rows and h must be positive");
  if (h % 8 || h > 8192) return fail(DOMINO_ERR_UNSUPPORTED, "h must be a multiple of 8 and at most 8192");
  NormFwdArgs a{};
  a.x = x; a.add1 = add1; a.add2 = add2; a.vec = vec; a.gamma = gamma; a.beta = beta; a.xsum = xsum; a.y = y;
  a.mean = rms ? nullptr : mean; a.rstd = rstd; a.rows = rows; a.h = h; a.rms = rms; a.eps = eps;
  HIP_TRY(norm_fwd_launch(a, as_stream(stream)), "norm forward launch");
  return DOMINO_OK;
}

size_t domino_norm_bwd_scratch_floats(int rows, int h) {
  if (rows <= 0 || h <= 0) return 0;
  return 2 * (size_t)norm_bwd_blocks(rows) * h;
}

int domino_norm_bwd(const void* ga, const void* gb, const void* x, const void* gamma,
                    const float* mean, const float* rstd, const void* dres, void* dx,
                    float* dgamma, float* dbeta, float* scratch,
                    int rows, int h, int rms, void* stream) {
  if (!ga || !x || !gamma || !rstd || !dx || !dgamma || !scratch) return fail(DOMINO_ERR_NULL_POINTER, "a required pointer is NULL");
  if (!rms && (!mean || !dbeta)) return fail(DOMINO_ERR_NULL_POINTER, "LayerNorm needs mean and dbeta");
  if (rows <= 0 || h <= 0) return fail(DOMINO_ERR_INVALID_ARG, "rows and h must be positive");
  if (h % 8 || h > 8192) return fail(DOMINO_ERR_UNSUPPORTED, "h must be a multiple of 8 and at most 8192");
  NormBwdArgs a{};
  a.ga = ga; a.gb = gb; a.x = x; a.gamma = gamma; a.mean = mean; a.rstd = rstd; a.dres = dres; a.dx = dx;
  const int nb = norm_bwd_blocks(rows);
  a.part_g = scratch; a.part_b = scratch + (size_t)nb * h; a.rows = rows; a.h = h; a.rms = rms;
  hipStream_t st = as_stream(stream);
  HIP_TRY(norm_bwd_launch(a, st), "norm backward launch");
  ColsumJobs jobs{};
  jobs.job[0] = {a.part_g, dgamma, nb, h, (long)h, 1, 0};
  jobs.job[1] = {a.part_b, dbeta, nb, h, (long)h, 1, 0};
  HIP_TRY(colsum_finish_jobs_launch(jobs, rms ? 1 : 2, 0, st), "norm gain / shift gradient");
  return DOMINO_OK;
}

static int check_attn(int64_t ld, int batch, int seq, int heads, int head_dim) {
  if (batch <= 0 || seq <= 0 || heads <= 0) return fail(DOMINO_ERR_INVALID_ARG, "batch, seq, heads must be positive");
  if (head_dim != 64 && head_dim != 80 && head_dim != 128) return fail(DOMINO_ERR_UNSUPPORTED, "head_dim %d not in {64, 80, 128}", head_dim);
  if (ld < 3L * heads * head_dim || ld % 8) return fail(DOMINO_ERR_INVALID_ARG, "ld must be a multiple of 8 and at least 3*heads*head_dim");
  if ((long)batch * seq * ld * 2 >= TWO_GIB) return fail(DOMINO_ERR_UNSUPPORTED, "qkv would reach 2 GiB");
  return DOMINO_OK;
}

int domino_attention_fwd(const void* qkv, int64_t ld, int batch, int seq, int heads, int head_dim,
                         void* ctx, float* lse, void* stream) {
  if (!qkv || !ctx || !lse) return fail(DOMINO_ERR_NULL_POINTER, "qkv, ctx or lse is NULL");
  TRY(check_attn(ld, batch, seq, heads, head_dim));
  AttnArgs a{};
  a.qkv = qkv; a.ld = ld; a.ctx = ctx; a.ld_ctx = (long)heads * head_dim; a.lse = lse;
  a.batch = batch; a.seq = seq; a.heads = heads; a.head_dim = head_dim; a.scale = 1.0f / sqrtf((float)head_dim);
  HIP_TRY(attention_fwd_launch(a, as_stream(stream)), "attention forward launch");
  return DOMINO_OK;
}

int domino_attention_bwd(const void* qkv, int64_t ld, const void* ctx, const void* dctx, const float* lse,
                         void* dqkv, float* dot, int batch, int seq, int heads, int head_dim, void* stream) {
  if (!qkv || !ctx || !dctx || !lse || !dqkv || !dot) return fail(DOMINO_ERR_NULL_POINTER, "a required pointer is NULL");
  TRY(check_attn(ld, batch, seq, heads, head_dim));
  AttnArgs a{};
  a.qkv = qkv; a.ld = ld; a.ctx = const_cast<void*>(ctx); a.ld_ctx = (long)heads * head_dim; a.dctx = dctx;
  a.lse = const_cast<float*>(lse); a.dot = dot; a.dqkv = dqkv;
  a.batch = batch; a.seq = seq; a.heads = heads; a.head_dim = head_dim; a.scale = 1.0f / sqrtf((float)head_dim);
  HIP_TRY(attention_bwd_launch(a, as_stream(stream)), "attention backward launch");
  return DOMINO_OK;
}

int domino_attention_bwd_rope(const void* qkv, int64_t ld, const void* ctx, const void* dctx, const float* lse,
                              void* dqkv, float* dot, int batch, int seq, int heads, int head_dim, float base, void* stream) {
  if (!qkv || !ctx || !dctx || !lse || !dqkv || !dot) return fail(DOMINO_ERR_NULL_POINTER, "a required pointer is NULL");
  TRY(check_attn(ld, batch, seq, heads, head_dim));
  if (!(base > 1.0f)) return fail(DOMINO_ERR_INVALID_ARG, "base must exceed 1");
  AttnArgs a{};
  a.qkv = qkv; a.ld = ld; a.ctx = const_cast<void*>(ctx); a.ld_ctx = (long)heads * head_dim; a.dctx = dctx;
  a.lse = const_cast<float*>(lse); a.dot = dot; a.dqkv = dqkv;
  a.batch = batch; a.seq = seq; a.heads = heads; a.head_dim = head_dim; a.scale = 1.0f / sqrtf((float)head_dim);
  a.rope = 1; a.rope_log2_base = log2f(base);
  HIP_TRY(attention_bwd_launch(a, as_stream(stream)), "attention backward launch");
  return DOMINO_OK;
}

int domino_rope(void* m, int64_t ld, int rows, int seq, int col0, int nblocks, int heads, int head_dim,
                float base, int inverse, void* stream) {
  if (!m) return fail(DOMINO_ERR_NULL_POINTER, "m is NULL");
  if (rows <= 0 || seq <= 0 || nblocks <= 0 || heads <= 0 || head_dim <= 0 || col0 < 0)
    return fail(DOMINO_ERR_INVALID_ARG, "rows, seq, nblocks, heads, head_dim must be positive");
  if (head_dim % 16 || col0 % 8 || ld % 8) return fail(DOMINO_ERR_UNSUPPORTED, "head_dim must be a multiple of 16, col0 and ld multiples of 8");
  if (col0 + (long)nblocks * heads * head_dim > ld) return fail(DOMINO_ERR_INVALID_ARG, "column blocks exceed ld");
  if (!(base > 1.0f)) return fail(DOMINO_ERR_INVALID_ARG, "base must exceed 1");
  HIP_TRY(rope_launch(m, ld, rows, seq, col0, nblocks, heads, head_dim, base, inverse, as_stream(stream)), "rope launch");
  return DOMINO_OK;
}

int domino_colsum(const void* g, int64_t ld, int rows, int n, float* out, int accumulate, float* scratch, void* stream) {
  if (!g || !out || !scratch) return fail(DOMINO_ERR_NULL_POINTER, "g, out or scratch is NULL");
  if (rows <= 0 || n <= 0) return fail(DOMINO_ERR_INVALID_ARG, "rows and n must be positive");
  if (n % 8 || ld % 8 || ld < n) return fail(DOMINO_ERR_UNSUPPORTED, "n and ld must be multiples of 8, ld >= n");
  hipStream_t st = as_stream(stream);
  HIP_TRY(colsum_partial_launch(g, ld, rows, n, scratch, st), "colsum launch");
  HIP_TRY(colsum_finish_launch(scratch, COLSUM_PARTS, n, out, accumulate, st), "colsum launch");
  return DOMINO_OK;
}

// ---- column sums without a scratch argument: for callers that cannot allocate -----------------------------------
// The first stage's partial rows live in a file-scope device array.  In host code the array's name is only a
// stand-in for the symbol: its device address is looked up once per device and only that address is handed to
// the kernels.
}  // extern "C"
namespace {
constexpr int COLSUM_STATIC_MAX_N = 8192;
static __device__ __align__(256) float scratch[COLSUM_PARTS * COLSUM_STATIC_MAX_N];     // 2 MiB on every GPU used
std::map<int, float*> g_scratch_ptr;       // per device: every GPU holds its own copy of the array at its own address

int static_scratch(float** ptr) {          // g_mutex held
  int dev = 0;
  HIP_TRY(hipGetDevice(&dev), "hipGetDevice");
  auto it = g_scratch_ptr.find(dev);
  if (it == g_scratch_ptr.end()) {
    float* p = nullptr;
    HIP_TRY(hipGetSymbolAddress(reinterpret_cast<void**>(&p), HIP_SYMBOL(scratch)), "hipGetSymbolAddress(scratch)");
    if (!p) return fail(DOMINO_ERR_HIP, "hipGetSymbolAddress(scratch) returned a null address");
    it = g_scratch_ptr.emplace(dev, p).first;
  }
  *ptr = it->second;
  return DOMINO_OK;
}
}  // namespace
extern "C" {

int domino_colsum_noalloc(const void* g, int64_t ld, int rows, int n, float* out, int accumulate, void* stream) {
  if (!g || !out) return fail(DOMINO_ERR_NULL_POINTER, "g or out is NULL");
  if (rows <= 0 || n <= 0) return fail(DOMINO_ERR_INVALID_ARG, "rows and n must be positive");
  if (n % 8 || ld % 8 || ld < n) return fail(DOMINO_ERR_UNSUPPORTED, "n and ld must be multiples of 8, ld >= n");
  if (n > COLSUM_STATIC_MAX_N)
    return fail(DOMINO_ERR_UNSUPPORTED, "n = %d exceeds the %d columns the library's own scratch holds; use domino_colsum "
                "with a scratch buffer of the caller's", n, COLSUM_STATIC_MAX_N);
  std::lock_guard<std::mutex> lock(g_mutex);
  float* part = nullptr;
  TRY(static_scratch(&part));
  hipStream_t st = as_stream(stream);
  // the first stage writes every one of its COLSUM_PARTS x n partial sums (zeros for row ranges past the end), so
  // nothing of an earlier call's contents is read and nothing has to be cleared
  HIP_TRY(colsum_partial_launch(g, ld, rows, n, part, st), "colsum launch");
  HIP_TRY(colsum_finish_launch(part, COLSUM_PARTS, n, out, accumulate, st), "colsum launch");
  return DOMINO_OK;
}

int domino_mfma_probe(const void* a, const void* b, float* out, int blocks, int iters, double* flops, void* stream) {
  return domino_mfma_probe_shape(DOMINO_MFMA_32x32x16, a, b, out, blocks, iters, flops, stream);
}
int domino_mfma_probe_shape(int shape, const void* a, const void* b, float* out, int blocks, int iters, double* flops, void* stream) {
  if (shape != DOMINO_MFMA_32x32x16 && shape != DOMINO_MFMA_16x16x32) return fail(DOMINO_ERR_INVALID_ARG, "MFMA shape %d is neither 32x32x16 (0) nor 16x16x32 (1)", shape);
  if (!a || !b || !out) return fail(DOMINO_ERR_NULL_POINTER, "a, b or out is NULL");
  if (blocks < 1 || blocks > 65536 || iters < 1 || iters > (1 << 24))
    return fail(DOMINO_ERR_INVALID_ARG, "blocks must lie in [1, 65536] and iters in [1, 2^24]");
  if (flops) *flops = (double)blocks * 4.0 * iters * MFMA_PROBE_FLOPS_PER_WAVE_ITER;
  HIP_TRY(mfma_probe_launch(shape, a, b, out, blocks, iters, as_stream(stream)), "mfma probe launch");
  return DOMINO_OK;
}

// ------------------------------------------------------------------------------------ instrumentation
int domino_profile_enable(int on) {
  std::lock_guard<std::mutex> lock(g_mutex);
  g_prof_on = on != 0;
  return DOMINO_OK;
}
int domino_profile_classes(void) { return PC_COUNT; }
const char* domino_profile_name(int cls) { return (cls >= 0 && cls < PC_COUNT) ? PROF_NAMES[cls] : ""; }

int domino_profile_read(int cls, double* total_ms, int* launches) {
  if (cls < 0 || cls >= PC_COUNT) return fail(DOMINO_ERR_INVALID_ARG, "class %d outside [0, %d)", cls, (int)PC_COUNT);
  if (!total_ms || !launches) return fail(DOMINO_ERR_NULL_POINTER, "total_ms or launches is NULL");
  std::lock_guard<std::mutex> lock(g_mutex);
  double tot = 0.0;
  int n = 0;
  for (auto& r : g_prof_recs) {
    if (r.cls != cls) continue;
    HIP_TRY(hipEventSynchronize(r.stop), "hipEventSynchronize");
    float ms = 0.0f;
    HIP_TRY(hipEventElapsedTime(&ms, r.start, r.stop), "hipEventElapsedTime");
    tot += ms;
    ++n;
  }
  *total_ms = tot;
  *launches = n;
  return DOMINO_OK;
}

int domino_profile_records(void) {
  std::lock_guard<std::mutex> lock(g_mutex);
  return (int)g_prof_recs.size();
}

int domino_profile_record(int index, int* cls, void** stream, double* start_ms, double* stop_ms) {
  if (!cls || !stream || !start_ms || !stop_ms) return fail(DOMINO_ERR_NULL_POINTER, "an output pointer is NULL");
  std::lock_guard<std::mutex> lock(g_mutex);
  if (index < 0 || index >= (int)g_prof_recs.size()) return fail(DOMINO_ERR_INVALID_ARG, "record %d outside [0, %d)", index, (int)g_prof_recs.size());
  const ProfRec& r = g_prof_recs[index];
  const ProfRec& first = g_prof_recs[0];
  HIP_TRY(hipEventSynchronize(first.start), "hipEventSynchronize");
  HIP_TRY(hipEventSynchronize(r.stop), "hipEventSynchronize");
  float a = 0.0f, b = 0.0f;
  HIP_TRY(hipEventElapsedTime(&a, first.start, r.start), "hipEventElapsedTime");
  HIP_TRY(hipEventElapsedTime(&b, first.start, r.stop), "hipEventElapsedTime");
  *cls = r.cls; *stream = r.stream; *start_ms = a; *stop_ms = b;
  return DOMINO_OK;
}

int domino_profile_reset(void) {
  std::lock_guard<std::mutex> lock(g_mutex);
  for (auto& r : g_prof_recs) { g_prof_free.push_back(r.start); g_prof_free.push_back(r.stop); }
  g_prof_recs.clear();
  return DOMINO_OK;
}

void domino_shutdown(void) {
  std::lock_guard<std::mutex> lock(g_mutex);
  for (auto& kv : g_pools)
    for (auto e : kv.second.events) (void)hipEventDestroy(e);
  g_pools.clear();
  g_pool = nullptr;
  for (auto& r : g_prof_recs) { (void)hipEventDestroy(r.start); (void)hipEventDestroy(r.stop); }
  g_prof_recs.clear();
  for (auto e : g_prof_free) (void)hipEventDestroy(e);
  g_prof_free.clear();
}

}  // extern "C"
