// Host-only check of the library's piece schedule (the host half of csrc/api.hip): this program links api.hip's host
// code against stand-ins for the HIP runtime and for the kernel launchers, lets the layer, parts and stack calls enqueue
// onto fake streams, and examines the recorded order of launches, event records and event waits:
//   - every launch is ordered after the call's first operation on streams[0] and before its last (fork and join);
//   - every stream other than streams[0] enters a call by waiting for an event recorded in that call (under HIP graph
//     capture this is how a stream joins the capture), and no wait refers to an event not yet recorded in the call;
//   - any two launches that touch overlapping memory, at least one of them writing, are ordered by stream order or by
//     a chain of events (the race check), over the buffers the launchers are handed; where products, a norm and column sums
//     share a launch, no two of these do;
//   - the weight gradients of a matrix, and the reductions of the vector gradients, are one launch over all rows, or
//     enqueued in slice order and ordered one after the other (the fixed accumulation order);
//   - the vector gradients sum partial rows that were written in this backward, and no launch writes over another's;
//   - over the parts of one backward every gradient is formed exactly once, whatever pool each part is handed and whichever
//     of them are captured or timed launch by launch;
//   - timing a step launch by launch changes none of its launches, and times each under its own step's name, what is held
//     back for a later launch with that launch;
//   - no call returns with work still held back;
//   - a captured call uses no event twice, and pools outside domino_capture_supported() are refused while capturing.
// Nothing here touches a GPU.  Exit status 0 = every expectation held.
#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <set>
#include <string>
#include <vector>

#include <hip/hip_runtime.h>

#include "../include/domino.h"
#include "../paper_2409_15241_amd/csrc/attention.h"
#include "../paper_2409_15241_amd/csrc/eltwise.h"
#include "../paper_2409_15241_amd/csrc/gemm.h"
#include "../paper_2409_15241_amd/csrc/norm.h"
#include "../paper_2409_15241_amd/csrc/probe.h"

// ------------------------------------------------------------------------------------------- the recorded schedule
struct Region {                      // rows x cols elements of `esz` bytes, `ld` elements from row to row
  const char* base; long ld; long rows, cols; int esz; bool write;
  enum Rows { PLAIN, NORM_SUMS, COLUMN_SUMS } partial = PLAIN;      // partial rows of vector gradients, and what leaves them
  int job = 0;                       // which of the products, norms and sums that share a launch touches it: these run side by side
};
struct Op {
  enum Kind { LAUNCH, RECORD, WAIT } kind;
  hipStream_t stream;
  void* event;                       // RECORD / WAIT
  std::string what;                  // LAUNCH: step name
  std::vector<Region> regions;
  struct Product { float* c; const char* a; long rows; int beta; };
  std::vector<Product> products;     // LAUNCH of weight gradients: the matrices they go into, the rows they contract over
  bool vec_reduce = false;           // LAUNCH of the vector-gradient reduction
};
static std::vector<Op> g_ops;
static bool g_per_slice = false;      // the configuration under test forms its weight gradients slice by slice
static bool g_merged = false;         // ... hands them over once per block (refused in a captured stack of several blocks)
static bool g_accumulate = false;
static long g_rows = 0;              // rows (batch x sequence) of the configuration under test
static bool g_capturing = false;
static int g_failures = 0;
static std::string g_case;

#define EXPECT(cond, ...)                                                        \
  do {                                                                           \
    if (!(cond)) {                                                               \
      std::printf("FAILED [%s] %s: ", g_case.c_str(), #cond);                   \
      std::printf(__VA_ARGS__);                                                  \
      std::printf("\n");                                                         \
      ++g_failures;                                                              \
    }                                                                            \
  } while (0)

static Region reg(const void* p, long ld, long rows, long cols, int esz, bool write) {
  return Region{static_cast<const char*>(p), ld, rows, cols, esz, write};
}
static Region partial_rows(Region::Rows kind, const void* p, long rows, long cols) {
  Region r = reg(p, cols, rows, cols, 4, true);
  r.partial = kind;
  return r;
}
static void launch(hipStream_t st, const char* what, std::vector<Region> r, std::vector<Op::Product> products = {}, bool vec = false) {
  Op o;
  o.kind = Op::LAUNCH; o.stream = st; o.event = nullptr; o.what = what; o.products = std::move(products); o.vec_reduce = vec;
  for (auto& x : r)
    if (x.base) o.regions.push_back(x);
  g_ops.push_back(std::move(o));
}

// ------------------------------------------------------------------------------------------- HIP runtime stand-ins
extern "C" {
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "stub"; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = reinterpret_cast<hipEvent_t>(new int(1)); /* 1: it can time */ return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { *e = reinterpret_cast<hipEvent_t>(new int(0)); return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { delete reinterpret_cast<int*>(e); return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 0.0f; return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
  Op o; o.kind = Op::RECORD; o.stream = s; o.event = e; g_ops.push_back(o); return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) {
  Op o; o.kind = Op::WAIT; o.stream = s; o.event = e; g_ops.push_back(o); return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* st) {
  *st = g_capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
  return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void*) { static float dummy[4]; *p = dummy; return hipSuccess; }
void** __hipRegisterFatBinary(const void*) { static void* h = nullptr; return &h; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterVar(void**, void*, char*, const char*, int, size_t, int, int) {}
}

// ------------------------------------------------------------------------------------------- launcher stand-ins
static const char* gemm_name(int layout, int epi) {
  if (layout == GEMM_NT) return epi == EPI_STORE ? "dgrad" : "dgrad+act'";
  return epi == EPI_STORE ? "gemm" : epi == EPI_ROPE ? "gemm+rope" : "gemm+act";
}
int norm_bwd_blocks(int rows) {
  const int want = (rows + NORM_BWD_ROWS - 1) / NORM_BWD_ROWS;
  return want < NORM_BWD_MAX_BLOCKS ? want : NORM_BWD_MAX_BLOCKS;
}
static std::vector<Region> norm_bwd_regions(const NormBwdArgs& a) {
  // one partial row per workgroup: slice_blocks of them for each slice
  const int slice_rows = a.slice_rows > 0 ? a.slice_rows : a.rows;
  const long nb = (long)(a.slice_blocks > 0 ? a.slice_blocks : norm_bwd_blocks(slice_rows)) * (a.rows / slice_rows);
  std::vector<Region> r = {reg(a.ga, a.h, a.rows, a.h, 2, false), reg(a.gb, a.h, a.rows, a.h, 2, false),
                           reg(a.x, a.h, a.rows, a.h, 2, false), reg(a.dres, a.h, a.rows, a.h, 2, false),
                           reg(a.mean, a.rows, 1, a.rows, 4, false), reg(a.rstd, a.rows, 1, a.rows, 4, false),
                           reg(a.dx, a.h, a.rows, a.h, 2, true)};
  for (float* part : {a.part_g, a.part_b, a.part_dres, a.part_dx}) r.push_back(partial_rows(Region::NORM_SUMS, part, nb, a.h));
  return r;
}
static std::vector<Region> colsum_regions(const ColsumPartial& c) {
  return {reg(c.g, c.ld, c.rows, c.n, 2, false), partial_rows(Region::COLUMN_SUMS, c.part, COLSUM_PARTS, c.n)};
}

// products held back by GemmArgs::join, and the stream of the first
static std::vector<GemmArgs> g_held;
static hipStream_t g_held_on;
static long g_range_launches = 0;     // launches over several contraction ranges, in all cases
static long g_norm_joins = 0, g_sum_joins = 0;      // Norm1 backwards and column sums launched with weight gradients, in all cases
static hipError_t launch_weight_gradients(const std::vector<GemmArgs>& held, hipStream_t st) {
  std::vector<Region> r, sums;
  std::vector<Op::Product> products;
  const int splits = held[0].splits > 1 ? held[0].splits : 1;
  long floats = 0;
  for (const GemmArgs& a : held) floats += (long)a.M * a.N;
  int job = 0;
  auto touch = [&](std::vector<Region>& to, Region x) { x.job = job; to.push_back(x); };
  for (const GemmArgs& a : held) {
    ++job;
    touch(r, reg(a.A, a.lda, a.K, a.M, 2, false));
    touch(r, reg(a.B, a.ldb, a.K, a.N, 2, false));
    touch(splits > 1 ? sums : r, reg(a.C, a.ldc, a.M, a.N, 4, true));
    products.push_back({static_cast<float*>(a.C), static_cast<const char*>(a.A), a.K, a.beta});
    EXPECT(a.K == held[0].K && a.beta == held[0].beta && a.splits == held[0].splits, "products of one launch differ in depth, ranges or accumulation");
    EXPECT(a.tail == held[0].tail, "products of one launch differ in what is launched with them");
  }
  if (held[0].tail) {                  // what t_tail holds: further workgroups of this launch
    EXPECT(t_tail.open && t_tail.stream == st, "weight gradients are launched with work that is not held back for their stream");
    const NormBwdArgs& norm = t_tail.norm;
    if (norm.rows) {
      EXPECT(splits == 1 && norm.h <= HeldTail::MAX_H && !norm.part_dres && !norm_streams(norm.rows, norm.h), "a norm is held back for a launch that does not take it");
      ++job;
      for (const Region& x : norm_bwd_regions(norm)) touch(r, x);
      ++g_norm_joins;
    }
    EXPECT(norm.rows || t_tail.nsums, "nothing is held back for a launch");
    for (int k = 0; k < t_tail.nsums; ++k, ++g_sum_joins) {
      ++job;
      for (const Region& x : colsum_regions(t_tail.sums[k])) touch(r, x);
    }
    t_tail.open = false;
  }
  if (splits == 1) { launch(st, "wgrad", r, products); return hipSuccess; }
  ++g_range_launches;
  EXPECT(held[0].split_ws != nullptr, "%d contraction ranges without memory for their sums", splits);
  r.push_back(reg(held[0].split_ws, floats, splits, floats, 4, true));
  launch(st, "wgrad ranges", r, products);
  sums.push_back(reg(held[0].split_ws, floats, splits, floats, 4, false));
  launch(st, "wgrad sum of ranges", sums);
  return hipSuccess;
}
hipError_t gemm_launch(int layout, int epi, const GemmArgs& a, int, hipStream_t st) {
  if (layout == GEMM_TN) {
    if (g_held.empty()) g_held_on = st;
    EXPECT(g_held_on == st, "products of one launch are handed over on two streams");
    if (!g_held.empty() && g_held.back().C == a.C) {       // the next rows of the same product
      GemmArgs& h = g_held.back();
      EXPECT(a.beta && static_cast<const char*>(h.A) + h.K * h.lda * 2 == a.A && static_cast<const char*>(h.B) + h.K * h.ldb * 2 == a.B,
             "a product into the same matrix does not continue the one before it");
      h.K += a.K;
    } else {
      EXPECT((int)g_held.size() < GEMM_GROUP, "more than %d products held back", GEMM_GROUP);
      g_held.push_back(a);
    }
    if (a.join) return hipSuccess;
    const std::vector<GemmArgs> held = std::move(g_held);
    g_held.clear();
    return launch_weight_gradients(held, st);
  }
  EXPECT(g_held.empty(), "a product is launched while weight gradients are held back");
  std::vector<Region> r;
  const bool glu = epi == EPI_SWIGLU || epi == EPI_DSWIGLU;
  r.push_back(reg(a.A, a.lda, a.M, a.K, 2, false));
  if (layout == GEMM_NT) r.push_back(reg(a.B, a.ldb, a.N, a.K, 2, false));
  else r.push_back(reg(a.B, a.ldb, a.K, epi == EPI_SWIGLU ? 2L * a.n_split : a.N, 2, false));
  r.push_back(reg(a.C, a.ldc, a.M, epi == EPI_DSWIGLU ? 2L * a.n_split : a.N, 2, true));
  if (a.bias) r.push_back(reg(a.bias, a.N, 1, a.N, 2, false));
  if (a.aux) r.push_back(reg(a.aux, a.ldaux, a.M, glu ? 2L * a.n_split : a.N, 2, epi == EPI_BIAS_GELU || epi == EPI_SWIGLU));
  if (a.add2) r.push_back(reg(a.add2, a.ldaux, a.M, a.N, 2, false));
  if (a.out2) r.push_back(reg(a.out2, a.ldaux, a.M, a.N, 2, true));
  launch(st, gemm_name(layout, epi), r);
  return hipSuccess;
}
hipError_t rope_launch(void* m, long ld, int rows, int, int col0, int nblocks, int heads, int d, float, int, hipStream_t st) {
  launch(st, "rope", {reg(static_cast<char*>(m) + 2L * col0, ld, rows, (long)nblocks * heads * d, 2, true)});
  return hipSuccess;
}
hipError_t norm_fwd_launch(const NormFwdArgs& a, hipStream_t st) {
  launch(st, "norm_fwd", {reg(a.x, a.h, a.rows, a.h, 2, false), reg(a.add1, a.h, a.rows, a.h, 2, false),
                          reg(a.add2, a.h, a.rows, a.h, 2, false), reg(a.xsum, a.h, a.rows, a.h, 2, true),
                          reg(a.y, a.h, a.rows, a.h, 2, true), reg(a.mean, a.rows, 1, a.rows, 4, true),
                          reg(a.rstd, a.rows, 1, a.rows, 4, true)});
  return hipSuccess;
}
hipError_t norm_bwd_launch(const NormBwdArgs& a, hipStream_t st) {
  if (a.join) {
    EXPECT(!t_tail.open, "a norm is held back over another");
    t_tail = HeldTail{a, {}, 0, st, true};
    return hipSuccess;
  }
  launch(st, "norm_bwd", norm_bwd_regions(a));
  return hipSuccess;
}
hipError_t attention_fwd_launch(const AttnArgs& a, hipStream_t st) {
  const long rows = (long)a.batch * a.seq;
  launch(st, "attn_fwd", {reg(a.qkv, a.ld, rows, 3L * a.heads * a.head_dim, 2, false),
                          reg(a.ctx, a.ld_ctx, rows, (long)a.heads * a.head_dim, 2, true),
                          reg(a.lse, rows * a.heads, 1, rows * a.heads, 4, true)});
  return hipSuccess;
}
hipError_t attention_bwd_launch(const AttnArgs& a, hipStream_t st) {
  const long rows = (long)a.batch * a.seq;
  launch(st, "attn_bwd", {reg(a.qkv, a.ld, rows, 3L * a.heads * a.head_dim, 2, false),
                          reg(a.ctx, a.ld_ctx, rows, (long)a.heads * a.head_dim, 2, false),
                          reg(a.dctx, a.ld_ctx, rows, (long)a.heads * a.head_dim, 2, false),
                          reg(a.lse, rows * a.heads, 1, rows * a.heads, 4, false),
                          reg(a.dot, rows * a.heads, 1, rows * a.heads, 4, true),
                          reg(a.dqkv, a.ld, rows, 3L * a.heads * a.head_dim, 2, true)});
  return hipSuccess;
}
hipError_t colsum_partial_launch(const void* g, long ld, int rows, int n, float* part, hipStream_t st) {
  const ColsumPartial c{g, ld, rows, n, part};
  if (t_tail.open && t_tail.stream == st && t_tail.nsums < COLSUM_MAX_HELD) {
    t_tail.sums[t_tail.nsums++] = c;
    return hipSuccess;
  }
  launch(st, "colsum_partial", colsum_regions(c));
  return hipSuccess;
}
// jobs held back by ColsumJobs::join, and their stream
static std::vector<ColsumJob> g_jobs;
static hipStream_t g_jobs_on;
hipError_t colsum_finish_jobs_launch(const ColsumJobs& jobs, int njobs, int accumulate, hipStream_t st) {
  if (g_jobs.empty()) {
    g_jobs.assign(jobs.job, jobs.job + njobs);
    g_jobs_on = st;
  } else {
    EXPECT(g_jobs_on == st && accumulate, "a continued reduction is on another stream, or does not accumulate");
    for (int k = 0; k < njobs; ++k) {
      bool found = false;
      for (ColsumJob& h : g_jobs)
        if (h.out == jobs.job[k].out) {
          found = h.part + h.nouter * h.ostride == jobs.job[k].part && h.nparts == jobs.job[k].nparts && h.ostride == jobs.job[k].ostride;
          h.nouter += jobs.job[k].nouter;
        }
      EXPECT(found, "a reduction does not continue one that is held back");
    }
  }
  if (jobs.join) return hipSuccess;
  std::vector<Region> r;
  for (const ColsumJob& j : g_jobs) {
    r.push_back(reg(j.out, j.n, 1, j.n, 4, true));
    for (int g = 0; g < j.nouter; ++g) r.push_back(reg(j.part + g * j.ostride, j.stride, j.nparts, j.n, 4, false));
  }
  g_jobs.clear();
  launch(st, "vector_gradients", r, {}, true);
  return hipSuccess;
}
hipError_t colsum_finish_launch(const float* part, int nparts, int n, float* out, int, hipStream_t st) {
  launch(st, "colsum_finish", {reg(part, n, nparts, n, 4, false), reg(out, n, 1, n, 4, true)});
  return hipSuccess;
}
hipError_t residual_out_launch(const void* x1, const void* a, const void* b, const void*, void* y, long n, int h, hipStream_t st) {
  launch(st, "residual_out", {reg(x1, h, n / h, h, 2, false), reg(a, h, n / h, h, 2, false), reg(b, h, n / h, h, 2, false),
                              reg(y, h, n / h, h, 2, true)});
  return hipSuccess;
}
hipError_t mfma_probe_launch(int, const void*, const void*, float*, int, int, hipStream_t) { return hipSuccess; }

// ------------------------------------------------------------------------------------------- the checks
static bool overlap(const Region& a, const Region& b) {
  const char *a0 = a.base, *a1 = a.base + ((a.rows - 1) * a.ld + a.cols) * a.esz;
  const char *b0 = b.base, *b1 = b.base + ((b.rows - 1) * b.ld + b.cols) * b.esz;
  if (a1 <= b0 || b1 <= a0) return false;
  if (a.ld == b.ld && a.esz == b.esz && a.ld > 0 && a.cols <= a.ld) {   // two windows of one matrix: compare rows and columns
    const long d = (b.base - a.base) / a.esz;                            // b's first element relative to a's
    const long pitch = a.ld;
    const long r = d >= 0 ? d / pitch : -((-d + pitch - 1) / pitch), c = d - r * pitch;   // 0 <= c < pitch
    if (c + b.cols <= pitch)                                             // b's rows do not wrap on a's grid
      return r < a.rows && r + b.rows > 0 && c < a.cols;                 // b's columns start at c >= 0: they meet a's [0, cols) iff c < cols
  }
  return true;                                                           // conservatively
}

struct Analysis {
  std::vector<std::vector<uint64_t>> before;   // before[i]: bitset of operations that happen before operation i
  bool hb(int a, int b) const { return (before[b][a >> 6] >> (a & 63)) & 1; }
};

static Analysis analyse(const std::vector<Op>& ops, int first) {
  const int n = (int)ops.size(), W = (n + 63) / 64;
  Analysis A;
  A.before.assign(n, std::vector<uint64_t>(W, 0));
  std::map<hipStream_t, int> last_on;          // last operation on a stream
  std::map<void*, int> record_of;              // latest record of an event
  for (int i = first; i < n; ++i) {
    auto add = [&](int j) {
      for (int w = 0; w < W; ++w) A.before[i][w] |= A.before[j][w];
      A.before[i][j >> 6] |= 1ull << (j & 63);
    };
    auto it = last_on.find(ops[i].stream);
    if (it != last_on.end()) add(it->second);
    if (ops[i].kind == Op::WAIT) {
      auto r = record_of.find(ops[i].event);
      EXPECT(r != record_of.end(), "operation %d waits for an event that this call has not recorded", i);
      if (r != record_of.end()) add(r->second);
    }
    if (ops[i].kind == Op::RECORD) record_of[ops[i].event] = i;
    last_on[ops[i].stream] = i;
  }
  return A;
}

// What the vector gradients take in, over operations [first, end) of g_ops that hold a whole backward: rows of partial sums
// written earlier, each by one launch only (two launches whose partial rows overlap would have outgrown their area).
static void check_partial_rows(int first) {
  std::vector<std::pair<const char*, const char*>> written;
  auto range = [](const Region& r) { return std::make_pair(r.base, r.base + ((r.rows - 1) * r.ld + r.cols) * r.esz); };
  for (int i = first; i < (int)g_ops.size(); ++i) {
    const Op& o = g_ops[i];
    if (o.kind != Op::LAUNCH) continue;
    for (const Region& r : o.regions)
      if (r.partial != Region::PLAIN) {
        const auto w = range(r);
        for (const auto& v : written)
          EXPECT(w.second <= v.first || v.second <= w.first, "launch %d (%s) writes over partial rows of another", i, o.what.c_str());
        written.push_back(w);
      }
    if (!o.vec_reduce) continue;
    for (const Region& r : o.regions) {
      if (r.write) continue;
      auto want = range(r);
      for (bool more = true; more && want.first < want.second;) {
        more = false;
        for (const auto& v : written)
          if (v.first <= want.first && want.first < v.second) { want.first = v.second; more = true; }
      }
      EXPECT(want.first >= want.second, "launch %d sums partial rows that nothing has written", i);
    }
  }
}

// one library call = operations [first, end) of g_ops
static void check_call(int first, hipStream_t s0, int p, bool capturing) {
  const int n = (int)g_ops.size();
  EXPECT(!t_tail.open && g_held.empty() && g_jobs.empty(), "the call returns with work still held back");
  if (first == n) return;
  const Analysis A = analyse(g_ops, first);
  int origin = -1, last0 = -1;
  for (int i = first; i < n; ++i)
    if (g_ops[i].stream == s0) { if (origin < 0) origin = i; last0 = i; }
  EXPECT(origin >= 0, "the call put nothing on streams[0]");
  std::set<hipStream_t> entered;
  std::set<void*> recorded;
  for (int i = first; i < n; ++i) {
    const Op& o = g_ops[i];
    if (o.stream != s0 && !entered.count(o.stream)) {
      entered.insert(o.stream);
      EXPECT(o.kind == Op::WAIT && A.hb(origin, i),
             "stream %p enters the call with operation %d, which is not a wait ordered after the call's start", (void*)o.stream, i);
    }
    if (o.kind == Op::RECORD) {
      if (capturing) EXPECT(!recorded.count(o.event), "event recorded twice inside one capture (operation %d)", i);
      recorded.insert(o.event);
    }
    if (o.kind != Op::LAUNCH) continue;
    EXPECT(i == origin || A.hb(origin, i) || o.stream == s0, "launch %d (%s) is not ordered after the call's start", i, o.what.c_str());
    EXPECT(i == last0 || A.hb(i, last0), "launch %d (%s) is not ordered before the call's end on streams[0]", i, o.what.c_str());
  }
  // races
  std::vector<int> L;
  for (int i = first; i < n; ++i)
    if (g_ops[i].kind == Op::LAUNCH) L.push_back(i);
  for (size_t x = 0; x < L.size(); ++x)
    for (size_t y = x + 1; y < L.size(); ++y) {
      const Op &a = g_ops[L[x]], &b = g_ops[L[y]];
      if (A.hb(L[x], L[y])) continue;
      for (const Region& ra : a.regions)
        for (const Region& rb : b.regions)
          if ((ra.write || rb.write) && overlap(ra, rb)) {
            EXPECT(false, "launches %d (%s) and %d (%s) touch the same memory unordered", L[x], a.what.c_str(), L[y], b.what.c_str());
            goto next_pair;
          }
    next_pair:;
    }
  for (int i : L) {                  // ... and inside a launch, between the jobs that share it
    const std::vector<Region>& r = g_ops[i].regions;
    bool clash = false;
    for (size_t x = 0; x < r.size(); ++x)
      for (size_t y = x + 1; y < r.size(); ++y) clash |= r[x].job != r[y].job && (r[x].write || r[y].write) && overlap(r[x], r[y]);
    EXPECT(!clash, "two jobs of launch %d (%s) touch the same memory", i, g_ops[i].what.c_str());
  }
  // fixed accumulation order: per matrix, and for the vector gradients, enqueue order = slice order, each ordered after the one before
  std::map<const void*, std::vector<int>> per_matrix, per_vector;     // keyed by the gradient tensor (one set per block of a stack)
  for (int i : L) {
    for (const Op::Product& w : g_ops[i].products) per_matrix[w.c].push_back(i);
    if (g_ops[i].vec_reduce)
      for (const Region& r : g_ops[i].regions)
        if (r.write) { per_vector[r.base].push_back(i); break; }
  }
  for (auto& kv : per_matrix) {
    // one launch over all rows, or slice by slice where the configuration asks for it; either way every row exactly once
    EXPECT((int)kv.second.size() == (g_per_slice ? p : 1), "%zu weight-gradient launches into one matrix for %d slices", kv.second.size(), p);
    auto product = [&](int i) {
      for (const Op::Product& w : g_ops[i].products)
        if (w.c == kv.first) return w;
      return Op::Product{};
    };
    long rows = 0;
    for (int i : kv.second) rows += product(i).rows;
    EXPECT(rows == g_rows, "the weight-gradient launches into one matrix contract over %ld rows of %ld", rows, g_rows);
    for (size_t k = 0; k < kv.second.size(); ++k)
      EXPECT(product(kv.second[k]).beta == (k > 0 || g_accumulate ? 1 : 0), "launch %zu into a matrix %s what it holds", k,
             product(kv.second[k]).beta ? "adds to" : "overwrites");
    // slice by slice: rows of slice k start k * Ms rows into the activation operand, so the k-th launch must be slice k's
    for (size_t k = 1; k < kv.second.size(); ++k) {
      EXPECT(A.hb(kv.second[k - 1], kv.second[k]), "weight gradients %d and %d into one matrix are not ordered", kv.second[k - 1], kv.second[k]);
      EXPECT(product(kv.second[k]).a > product(kv.second[k - 1]).a, "weight gradients into one matrix are not enqueued in slice order");
    }
  }
  for (auto& kv : per_vector) {
    EXPECT((int)kv.second.size() == (g_per_slice ? p : 1), "%zu vector-gradient reductions for %d slices", kv.second.size(), p);
    long groups = 0;                 // every slice's partial rows exactly once (read off the launch's first vector, a norm gain)
    for (int i : kv.second) {
      const std::vector<Region>& r = g_ops[i].regions;
      for (size_t k = 1; k < r.size() && !r[k].write; ++k) ++groups;
    }
    EXPECT(groups == p, "the vector-gradient reductions of a block sum %ld slices' partial rows of %d", groups, p);
    for (size_t k = 1; k < kv.second.size(); ++k)
      EXPECT(A.hb(kv.second[k - 1], kv.second[k]), "vector-gradient reductions %d and %d are not ordered", kv.second[k - 1], kv.second[k]);
  }
}

// ------------------------------------------------------------------------------------------- driving the library
struct Buffers {                                    // addresses only: one arena for all cases, never written or read
  char* mem;
  size_t size, used = 0;
  explicit Buffers(size_t bytes) : size(bytes) {
    static char* arena = static_cast<char*>(std::malloc(bytes));
    mem = arena;
  }
  void* take(size_t bytes) {
    void* p = mem + used;
    used += (bytes + 255) / 256 * 256;
    if (used > size) { std::printf("arena too small\n"); std::exit(2); }
    return p;
  }
};

// Blocks of three sizes: a small one, which keeps to one stream; one of few weight-gradient tiles and many rows, whose
// gradients are formed over several contraction ranges; one so wide that row groups run side by side and the weight
// gradients beside them.
enum { SMALL, DEEP, WIDE };
static const int SIZES[] = {SMALL, DEEP, WIDE};
static const char* const SIZE_NAMES[] = {"", "deep ", "wide "};
static int g_size = SMALL;

static domino_cfg make_cfg(int arch, int p, int q, bool per_slice) {
  domino_cfg c{};
  c.wgrad_per_slice = per_slice ? 1 : 0;
  c.hidden = 256; c.heads = 4; c.tp = 2; c.rank = 1; c.p = p; c.q = q; c.batch = 8; c.seq = 64;
  c.ffn = arch == DOMINO_ARCH_LLAMA ? 704 : 1024;
  if (g_size == DEEP) { c.hidden = 2560; c.heads = 32; c.tp = 8; c.seq = 2048; c.ffn = 10240; }
  if (g_size == WIDE) { c.hidden = 4096; c.heads = 32; c.tp = 4; c.seq = 1024; c.ffn = 16384; }
  c.arch = arch; c.gelu_tanh = 1; c.norm_eps = 1e-5f; c.rope_base = 10000.0f;
  return c;
}

struct Layer {
  domino_params P{};
  domino_grads G{};
  void *attn_others, *mlp_others, *attn_partial, *mlp_partial, *y, *saved, *dln2_others, *dln1_others, *dln2_partial, *dln1_partial;
};

static Layer make_layer(Buffers& B, const domino_cfg& c) {
  Layer L;
  const size_t h = c.hidden, hl = h / c.tp, fl = c.ffn / c.tp, up = fl * (c.arch == DOMINO_ARCH_LLAMA ? 2 : 1);
  const size_t act = (size_t)c.batch * c.seq * h * 2;
  const bool gpt = c.arch == DOMINO_ARCH_GPT;
  L.P.norm1_g = B.take(h * 2); L.P.norm2_g = B.take(h * 2);
  L.P.w_qkv = B.take(h * 3 * hl * 2); L.P.w_o = B.take(hl * h * 2); L.P.w_up = B.take(h * up * 2); L.P.w_down = B.take(fl * h * 2);
  L.G.norm1_g = (float*)B.take(h * 4); L.G.norm2_g = (float*)B.take(h * 4);
  L.G.w_qkv = (float*)B.take(h * 3 * hl * 4); L.G.w_o = (float*)B.take(hl * h * 4);
  L.G.w_up = (float*)B.take(h * up * 4); L.G.w_down = (float*)B.take(fl * h * 4);
  if (gpt) {
    L.P.norm1_b = B.take(h * 2); L.P.norm2_b = B.take(h * 2); L.P.b_qkv = B.take(3 * hl * 2); L.P.b_o = B.take(h * 2);
    L.P.b_up = B.take(fl * 2); L.P.b_down = B.take(h * 2);
    L.G.norm1_b = (float*)B.take(h * 4); L.G.norm2_b = (float*)B.take(h * 4); L.G.b_qkv = (float*)B.take(3 * hl * 4);
    L.G.b_o = (float*)B.take(h * 4); L.G.b_up = (float*)B.take(fl * 4); L.G.b_down = (float*)B.take(h * 4);
  }
  L.attn_others = B.take(act); L.mlp_others = B.take(act); L.attn_partial = B.take(act); L.mlp_partial = B.take(act);
  L.y = B.take(act); L.saved = B.take(domino_saved_bytes(&c));
  L.dln2_others = B.take(act); L.dln1_others = B.take(act); L.dln2_partial = B.take(act); L.dln1_partial = B.take(act);
  return L;
}

static void run_case(int arch, int p, int q, int nstreams, bool capturing, int nlayers, bool parts, bool per_slice = false) {
  char name[160];
  std::snprintf(name, sizeof(name), "%s%s p=%d q=%d streams=%d%s layers=%d%s", SIZE_NAMES[g_size], arch ? "llama" : "gpt", p, q, nstreams,
                capturing ? " capturing" : "", nlayers, parts ? (per_slice ? " parts per-slice" : " parts") : (per_slice ? " per-slice" : ""));
  g_case = name;
  const domino_cfg c = make_cfg(arch, p, q, per_slice);
  g_merged = p > 2 && !per_slice;
  g_per_slice = per_slice;
  g_accumulate = false;
  g_rows = (long)c.batch * c.seq;
  if (domino_validate_cfg(&c) != DOMINO_OK) { EXPECT(false, "configuration rejected: %s", domino_last_error()); return; }
  Buffers B((size_t)12 << 30);
  std::vector<Layer> layers;
  for (int l = 0; l < nlayers; ++l) layers.push_back(make_layer(B, c));
  const size_t act = (size_t)c.batch * c.seq * c.hidden * 2;
  void* x = B.take(act);
  void* dy = B.take(act);
  void* dx = B.take(act);
  const size_t wsb = nlayers > 1 ? domino_stack_workspace_bytes(&c, nlayers) : domino_workspace_bytes(&c);
  void* ws = B.take(wsb);
  std::vector<void*> streams;
  for (int k = 0; k < nstreams; ++k) streams.push_back(reinterpret_cast<void*>((uintptr_t)0x1000 * (k + 1)));
  hipStream_t s0 = static_cast<hipStream_t>(streams[0]);
  g_capturing = capturing;
  const bool ok_pool = !capturing || domino_capture_supported(nstreams, p);
  auto call = [&](int rc, const char* what) {
    if (ok_pool) EXPECT(rc == DOMINO_OK, "%s returned %d: %s", what, rc, domino_last_error());
    else EXPECT(rc == DOMINO_ERR_UNSUPPORTED, "%s under capture with an unsupported pool returned %d", what, rc);
  };
  g_ops.clear();
  if (nlayers == 1) {
    Layer& L = layers[0];
    if (!parts) {
      int first = (int)g_ops.size();
      call(domino_layer_fwd(&c, &L.P, x, L.attn_others, L.mlp_others, L.attn_partial, L.mlp_partial, L.y, L.saved, ws, wsb,
                            streams.data(), nstreams), "domino_layer_fwd");
      if (!ok_pool) { EXPECT(g_ops.empty(), "a refused call enqueued %zu operations", g_ops.size()); g_capturing = false; return; }
      if (!capturing) check_call(first, s0, p, false);
      const int mid = (int)g_ops.size();
      call(domino_layer_bwd(&c, &L.P, L.saved, x, dy, L.dln2_others, L.dln1_others, L.dln2_partial, L.dln1_partial, dx, &L.G, 0,
                            ws, wsb, streams.data(), nstreams), "domino_layer_bwd");
      // a capture holds the forward and the backward: checked as one unit (events must not repeat across the two calls)
      check_call(capturing ? first : mid, s0, p, capturing);
      check_partial_rows(mid);
    } else {
      const int fparts[2] = {DOMINO_FWD_ATTN, DOMINO_FWD_MLP};
      for (int k = 0; k < 2; ++k) {
        const int first = (int)g_ops.size();
        call(domino_layer_fwd_parts(&c, &L.P, x, L.attn_others, L.mlp_others, L.attn_partial, L.mlp_partial, L.y, L.saved, ws, wsb,
                                    streams.data(), nstreams, fparts[k]), "domino_layer_fwd_parts");
        check_call(first, s0, p, false);
      }
      const int bparts[3] = {DOMINO_BWD_MLP, DOMINO_BWD_ATTN, DOMINO_BWD_NORM1};
      for (int k = 0; k < 3; ++k) {
        const int first = (int)g_ops.size();
        call(domino_layer_bwd_parts(&c, &L.P, L.saved, x, dy, L.dln2_others, L.dln1_others, L.dln2_partial, L.dln1_partial, dx, &L.G,
                                    0, ws, wsb, streams.data(), nstreams, bparts[k]), "domino_layer_bwd_parts");
        check_call(first, s0, p, false);
      }
      check_partial_rows(0);
    }
  } else {
    std::vector<domino_params> P;
    std::vector<domino_grads> G;
    std::vector<domino_stack_fwd_io> fio;
    std::vector<domino_stack_bwd_io> bio;
    for (int l = 0; l < nlayers; ++l) {
      Layer& L = layers[l];
      P.push_back(L.P); G.push_back(L.G);
      fio.push_back({L.attn_others, L.mlp_others, L.attn_partial, L.mlp_partial, L.y, L.saved});
      bio.push_back({l == 0 ? x : layers[l - 1].y, L.saved, L.dln2_others, L.dln1_others, L.dln2_partial, L.dln1_partial});
    }
    int first = (int)g_ops.size();
    call(domino_stack_fwd(&c, nlayers, P.data(), x, fio.data(), ws, wsb, streams.data(), nstreams), "domino_stack_fwd");
    if (!ok_pool) { g_capturing = false; return; }
    if (!capturing) check_call(first, s0, p, false);
    const int mid = (int)g_ops.size();
    const int rc = domino_stack_bwd(&c, nlayers, P.data(), dy, bio.data(), dx, G.data(), 0, ws, wsb, streams.data(), nstreams);
    if (capturing && g_merged && nlayers > 1) {   // merged weight gradients over several blocks: not under capture
      EXPECT(rc == DOMINO_ERR_UNSUPPORTED, "a captured stack backward with merged weight gradients returned %d", rc);
      EXPECT((int)g_ops.size() == mid, "a refused call enqueued %zu operations", g_ops.size() - mid);
      check_call(first, s0, p, true);             // the captured forward on its own
    } else {
      call(rc, "domino_stack_bwd");
      check_call(capturing ? first : mid, s0, p, capturing);
      check_partial_rows(mid);
    }
  }
  g_capturing = false;
}

// One backward in its three parts, each call in a situation of its own (the pool it is handed, whether it is captured,
// whether per-launch timing is on): whatever the situations, over the whole backward every gradient is formed exactly once.
struct Situation { int nstreams; bool capturing, timed; };
static int run_mixed_parts(int arch, int p, int accumulate) {
  const Situation some[] = {{1, false, false}, {4, false, false}, {4, true, false}, {4, false, true}};
  const int bparts[3] = {DOMINO_BWD_MLP, DOMINO_BWD_ATTN, DOMINO_BWD_NORM1};
  const domino_cfg c = make_cfg(arch, p, 1, false);
  g_merged = p > 2;
  g_per_slice = false;
  g_accumulate = accumulate != 0;
  g_rows = (long)c.batch * c.seq;
  Buffers B((size_t)12 << 30);
  Layer L = make_layer(B, c);
  const size_t act = (size_t)c.batch * c.seq * c.hidden * 2, wsb = domino_workspace_bytes(&c);
  void *x = B.take(act), *dy = B.take(act), *dx = B.take(act), *ws = B.take(wsb);
  void* streams[4];
  for (int k = 0; k < 4; ++k) streams[k] = reinterpret_cast<void*>((uintptr_t)0x1000 * (k + 1));
  int cases = 0;
  for (int sit = 0; sit < 64; ++sit, ++cases) {
    const Situation at[3] = {some[sit / 16], some[sit / 4 % 4], some[sit % 4]};
    auto kind = [](const Situation& s) { return s.capturing ? " captured" : s.timed ? " timed" : ""; };
    char name[160];
    std::snprintf(name, sizeof(name), "%s%s p=%d parts on %d%s, %d%s, %d%s streams", SIZE_NAMES[g_size], arch ? "llama" : "gpt", p,
                  at[0].nstreams, kind(at[0]), at[1].nstreams, kind(at[1]), at[2].nstreams, kind(at[2]));
    g_case = name;
    g_ops.clear();
    for (int k = 0; k < 3; ++k) {
      const int first = (int)g_ops.size();
      g_capturing = at[k].capturing;
      domino_profile_enable(at[k].timed);
      const int rc = domino_layer_bwd_parts(&c, &L.P, L.saved, x, dy, L.dln2_others, L.dln1_others, L.dln2_partial, L.dln1_partial, dx,
                                            &L.G, accumulate, ws, wsb, streams, at[k].nstreams, bparts[k]);
      g_capturing = false;
      domino_profile_enable(0);
      EXPECT(rc == DOMINO_OK, "part %d returned %d: %s", bparts[k], rc, domino_last_error());
      check_call(first, static_cast<hipStream_t>(streams[0]), p, at[k].capturing);
    }
    const float* const vecs[] = {L.G.norm1_g, L.G.norm1_b, L.G.norm2_g, L.G.norm2_b, L.G.b_qkv, L.G.b_o, L.G.b_up, L.G.b_down};
    const char* const names[] = {"norm1_g", "norm1_b", "norm2_g", "norm2_b", "b_qkv", "b_o", "b_up", "b_down"};
    for (int v = 0; v < 8; ++v) {
      if (!vecs[v]) continue;
      long summed = 0;               // sets of partial rows that the vector's reductions take in
      for (const Op& o : g_ops)
        for (size_t r = 0; o.vec_reduce && r < o.regions.size(); ++r)
          if (o.regions[r].write && o.regions[r].base == reinterpret_cast<const char*>(vecs[v]))
            for (size_t k = r + 1; k < o.regions.size() && !o.regions[k].write; ++k) ++summed;
      const bool by_group = v == 4 || v == 6;          // column sums: as many sets as were made
      long want = p;
      if (by_group) {
        want = 0;
        for (const Op& o : g_ops)
          for (const Region& r : o.regions)
            if (r.partial == Region::COLUMN_SUMS && r.cols == (v == 4 ? 3L * c.hidden / c.tp : (long)c.ffn / c.tp)) ++want;
      }
      EXPECT(summed == want, "%s takes in %ld sets of partial rows of %ld over the three parts", names[v], summed, want);
    }
    check_partial_rows(0);
    const float* const mats[] = {L.G.w_qkv, L.G.w_o, L.G.w_up, L.G.w_down};
    for (const float* m : mats) {
      long rows = 0;
      for (const Op& o : g_ops)
        for (const Op::Product& w : o.products)
          if (w.c == m) rows += w.rows;
      EXPECT(rows == g_rows, "a matrix' weight gradient contracts over %ld rows of %ld over the three parts", rows, g_rows);
    }
  }
  return cases;
}

// The step class that a launch's record has to carry: products by their place in the block, the rest by what they are.
static bool class_fits(const std::string& cls, const std::string& what) {
  auto starts = [&](const char* s) { return cls.rfind(s, 0) == 0; };
  if (what == "colsum_partial" || what == "vector_gradients") return cls == "colsum";
  if (what.rfind("gemm", 0) == 0) return starts("gemm_");
  if (what.rfind("dgrad", 0) == 0) return starts("dgrad_");
  if (what.rfind("wgrad", 0) == 0) return starts("wgrad_");
  return cls == what;        // norm_fwd, norm_bwd, attn_fwd, attn_bwd, rope, residual_out
}

// Per-launch timing adds event records and nothing else: the launches of a timed step are those of an untimed one, and
// every record carries the class of the launches that it brackets.
static void run_timed(int arch, int p, int nstreams) {
  char name[160];
  std::snprintf(name, sizeof(name), "%s%s p=%d streams=%d timed", SIZE_NAMES[g_size], arch ? "llama" : "gpt", p, nstreams);
  g_case = name;
  const domino_cfg c = make_cfg(arch, p, 2, false);
  Buffers B((size_t)12 << 30);
  Layer L = make_layer(B, c);
  const size_t act = (size_t)c.batch * c.seq * c.hidden * 2, wsb = domino_workspace_bytes(&c);
  void *x = B.take(act), *dy = B.take(act), *dx = B.take(act), *ws = B.take(wsb);
  void* streams[8];
  for (int k = 0; k < 8; ++k) streams[k] = reinterpret_cast<void*>((uintptr_t)0x1000 * (k + 1));
  std::vector<Op> seen[2];
  domino_profile_reset();
  for (int timed = 0; timed < 2; ++timed) {
    g_ops.clear();
    domino_profile_enable(timed);
    int rc = domino_layer_fwd(&c, &L.P, x, L.attn_others, L.mlp_others, L.attn_partial, L.mlp_partial, L.y, L.saved, ws, wsb, streams, nstreams);
    EXPECT(rc == DOMINO_OK, "domino_layer_fwd returned %d: %s", rc, domino_last_error());
    rc = domino_layer_bwd(&c, &L.P, L.saved, x, dy, L.dln2_others, L.dln1_others, L.dln2_partial, L.dln1_partial, dx, &L.G, 0, ws, wsb,
                          streams, nstreams);
    EXPECT(rc == DOMINO_OK, "domino_layer_bwd returned %d: %s", rc, domino_last_error());
    domino_profile_enable(0);
    EXPECT((domino_profile_records() > 0) == (timed == 1), "%d launches were timed", domino_profile_records());
    for (const Op& o : g_ops)
      if (o.kind == Op::LAUNCH) seen[timed].push_back(o);
    // the timing events of a stream come in pairs, and every pair brackets launches
    std::map<hipStream_t, int> open;           // launches since the start event, or -1 outside a pair
    std::map<hipStream_t, std::vector<std::string>> inside;
    int record = 0;
    for (const Op& o : g_ops) {
      int& n = open.emplace(o.stream, -1).first->second;
      if (o.kind == Op::LAUNCH && n >= 0) { ++n; inside[o.stream].push_back(o.what); }
      if (o.kind == Op::LAUNCH && timed) EXPECT(n > 0, "a launch (%s) is not timed", o.what.c_str());
      if (o.kind != Op::RECORD || *static_cast<int*>(o.event) != 1) continue;
      EXPECT(n != 0, "two timing events with nothing between them");
      if (n > 0) {                             // the pair's second event: records are kept in the order in which pairs close
        int cls = -1;
        void* on = nullptr;
        double from, to;
        EXPECT(domino_profile_record(record++, &cls, &on, &from, &to) == DOMINO_OK && on == o.stream, "record %d is of another stream", record - 1);
        for (const std::string& what : inside[o.stream])
          EXPECT(class_fits(domino_profile_name(cls), what), "a launch (%s) is timed as %s", what.c_str(), domino_profile_name(cls));
        inside[o.stream].clear();
      }
      n = n < 0 ? 0 : -1;
    }
  }
  domino_profile_reset();
  EXPECT(seen[0].size() == seen[1].size(), "%zu launches with timing, %zu without", seen[1].size(), seen[0].size());
  for (size_t i = 0; i < seen[0].size() && i < seen[1].size(); ++i) {
    const Op &a = seen[0][i], &b = seen[1][i];
    bool same = a.what == b.what && a.stream == b.stream && a.regions.size() == b.regions.size();
    for (size_t r = 0; same && r < a.regions.size(); ++r)
      same = a.regions[r].base == b.regions[r].base && a.regions[r].rows == b.regions[r].rows && a.regions[r].cols == b.regions[r].cols;
    EXPECT(same, "launch %zu differs with timing (%s, %s)", i, a.what.c_str(), b.what.c_str());
  }
}

// The note about hardware queues speaks of the streams that a call uses, not of the pool's size: a small block uses one,
// whatever the pool; a wide block's backward three, two groups' and the weight gradients', which the runtime's default of
// four queues serves beside the null stream.
static void run_queue_note() {
  g_case = "hardware-queue note";
  auto note_after = [](int size, const char* queues) -> std::string {
    g_size = size;
    const domino_cfg c = make_cfg(DOMINO_ARCH_GPT, 4, 1, false);
    Buffers B((size_t)12 << 30);
    Layer L = make_layer(B, c);
    const size_t act = (size_t)c.batch * c.seq * c.hidden * 2, wsb = domino_workspace_bytes(&c);
    void *x = B.take(act), *dy = B.take(act), *dx = B.take(act), *ws = B.take(wsb);
    void* streams[8];
    for (int k = 0; k < 8; ++k) streams[k] = reinterpret_cast<void*>((uintptr_t)0x1000 * (k + 1));
    if (queues) setenv("GPU_MAX_HW_QUEUES", queues, 1); else unsetenv("GPU_MAX_HW_QUEUES");
    EXPECT(domino_layer_bwd(&c, &L.P, L.saved, x, dy, L.dln2_others, L.dln1_others, L.dln2_partial, L.dln1_partial, dx, &L.G, 0, ws, wsb,
                            streams, 8) == DOMINO_OK, "domino_layer_bwd: %s", domino_last_error());
    unsetenv("GPU_MAX_HW_QUEUES");
    return domino_last_warning();
  };
  std::string note = note_after(SMALL, "2");
  EXPECT(note.empty(), "a block on one stream gets the note: %s", note.c_str());
  for (const char* enough : {(const char*)nullptr, "4", "8"}) {
    note = note_after(WIDE, enough);
    EXPECT(note.empty(), "three streams with enough queues get the note: %s", note.c_str());
  }
  note = note_after(WIDE, "3");
  EXPECT(note.find("GPU_MAX_HW_QUEUES") != std::string::npos && note.find(">= 4") != std::string::npos, "three streams on three queues: '%s'", note.c_str());
}

int main() {
  run_queue_note();          // before any other call: the note is made once in a process
  int cases = 0;
  for (int size : SIZES)
  for (int arch : {DOMINO_ARCH_GPT, DOMINO_ARCH_LLAMA})
    for (int p : {1, 2, 4, 8})
      for (int q : {1, 2})
        for (int ns = 1; ns <= 8; ++ns) {
          g_size = size;
          run_case(arch, p, q, ns, false, 1, false); ++cases;
          run_case(arch, p, q, ns, true, 1, false); ++cases;
          // four blocks: the tensors handed from block to block, taken in turn, come round again
          if (q == 2) { run_case(arch, p, q, ns, false, 4, false); run_case(arch, p, q, ns, true, 4, false); cases += 2; }
          if (q == 1) { run_case(arch, p, q, ns, false, 1, true); ++cases; }
          if (p > 2 && q == 2) {      // the slice-by-slice weight gradients of Sec. 4.1.2 for more than two slices
            run_case(arch, p, q, ns, false, 1, false, true); run_case(arch, p, q, ns, true, 1, false, true);
            run_case(arch, p, q, ns, false, 4, false, true); run_case(arch, p, q, ns, true, 4, false, true);
            cases += 4;
          }
          if (p == 4 && q == 1) { run_case(arch, p, q, ns, false, 1, true, true); ++cases; }
        }
  for (int size : SIZES)
    for (int arch : {DOMINO_ARCH_GPT, DOMINO_ARCH_LLAMA})
      for (int p : {1, 2, 4})
        for (int accumulate : {0, 1}) {
          g_size = size;
          cases += run_mixed_parts(arch, p, accumulate);
        }
  for (int size : SIZES)
    for (int arch : {DOMINO_ARCH_GPT, DOMINO_ARCH_LLAMA})
      for (int p : {1, 2, 4, 8})
        for (int ns : {1, 2, 4}) { g_size = size; run_timed(arch, p, ns); ++cases; }
  EXPECT(g_range_launches > 0, "no case formed its weight gradients over several contraction ranges");
  EXPECT(g_norm_joins > 0 && g_sum_joins > 0, "no case launched a Norm1 backward (%ld) or column sums (%ld) with its weight gradients", g_norm_joins, g_sum_joins);
  // the check must be able to fail: two launches on different fake streams that write one buffer, no event between them
  {
    g_case = "planted race";
    g_ops.clear();
    static char buf[4096];
    const int before = g_failures;
    hipStream_t a = reinterpret_cast<hipStream_t>((uintptr_t)0x1000), b = reinterpret_cast<hipStream_t>((uintptr_t)0x2000);
    hipEvent_t e;
    (void)hipEventCreateWithFlags(&e, 0);
    (void)hipEventRecord(e, a);
    (void)hipStreamWaitEvent(b, e, 0);
    launch(a, "writer 1", {reg(buf, 64, 8, 64, 2, true)});
    launch(b, "writer 2", {reg(buf + 64, 64, 8, 32, 2, true)});
    (void)hipEventRecord(e, b);
    (void)hipStreamWaitEvent(a, e, 0);
    std::printf("(the next FAILED line is the planted race being found)\n");
    check_call(0, a, 1, false);
    if (g_failures == before + 1) g_failures = before;
    else { std::printf("the race check did not find the planted race\n"); ++g_failures; }
    // ... and two windows of one matrix that do not meet (different column ranges) are not a race
    g_ops.clear();
    (void)hipEventRecord(e, a);
    (void)hipStreamWaitEvent(b, e, 0);
    launch(a, "piece 0", {reg(buf, 64, 8, 32, 2, true)});
    launch(b, "piece 1", {reg(buf + 64, 64, 8, 32, 2, true)});
    (void)hipEventRecord(e, b);
    (void)hipStreamWaitEvent(a, e, 0);
    check_call(0, a, 1, false);
    // two jobs of one launch, the second writing a row that the first reads
    g_ops.clear();
    const int jobs_before = g_failures;
    Region second = reg(buf + 2 * 64 * 2, 64, 1, 64, 2, true);
    second.job = 1;
    launch(a, "wgrad", {reg(buf, 64, 8, 64, 2, false), second});
    std::printf("(the next FAILED line is the planted clash inside a launch being found)\n");
    check_call(0, a, 1, false);
    if (g_failures == jobs_before + 1) g_failures = jobs_before;
    else { std::printf("the race check did not find the planted clash inside a launch\n"); ++g_failures; }
    // the check of partial rows must be able to fail, too: a reduction of four rows where three were written
    g_ops.clear();
    const int had = g_failures;
    launch(a, "colsum_partial", {partial_rows(Region::COLUMN_SUMS, buf, 3, 16)});
    launch(a, "vector_gradients", {reg(buf + 2048, 16, 1, 16, 4, true), reg(buf, 16, 4, 16, 4, false)}, {}, true);
    std::printf("(the next FAILED line is the planted unwritten row being found)\n");
    check_partial_rows(0);
    if (g_failures == had + 1) g_failures = had;
    else { std::printf("the check of partial rows did not find the planted one\n"); ++g_failures; }
  }
  domino_shutdown();
  std::printf(g_failures ? "host schedule driver: %d expectation(s) failed over %d cases\n" : "host schedule driver: ok (%d cases)\n",
              g_failures ? g_failures : cases, cases);
  return g_failures ? 1 : 0;
}
