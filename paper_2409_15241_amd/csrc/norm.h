// Internal launcher interface of the normalisation and column-reduction kernels (see norm.hip).
#pragma once
#include <hip/hip_runtime.h>

constexpr int NORM_BWD_MAX_BLOCKS = 256;   // one partial row of d gamma / d beta per workgroup
constexpr int NORM_BWD_ROWS = 16;          // most rows per workgroup until the block limit is reached
constexpr int COLSUM_PARTS = 64;           // row ranges of the first column-sum stage

struct NormFwdArgs {
  const void* x;          // bf16 [rows, h]
  const void* add1;       // bf16 [rows, h] or null   (a partial sum to add before normalising)
  const void* add2;       // bf16 [rows, h] or null   (the other ranks' sum)
  const void* vec;        // bf16 [h] or null          (a bias added to every row)
  const void* gamma;      // bf16 [h]
  const void* beta;       // bf16 [h] or null
  void* xsum;             // bf16 [rows, h] or null: x + add1 + add2 + vec
  void* y;                // bf16 [rows, h]
  float* mean;            // fp32 [rows] or null (unused for RMSNorm)
  float* rstd;            // fp32 [rows]
  int rows, h, rms;
  float eps;
};

struct NormBwdArgs {
  const void* ga;         // bf16 [rows, h]: gradient w.r.t. the norm output (this rank's partial)
  const void* gb;         // bf16 [rows, h] or null: the other ranks' sum, added to ga
  const void* x;          // bf16 [rows, h]: the norm input
  const void* gamma;      // bf16 [h]
  const float* mean;      // fp32 [rows] (LayerNorm only)
  const float* rstd;      // fp32 [rows]
  const void* dres;       // bf16 [rows, h] or null: gradient arriving over the residual branch
  void* dx;               // bf16 [rows, h] = dres + NormBwd(ga + gb)
  // partial column sums: slice_blocks rows of h for each slice of slice_rows rows; every workgroup of the launch leaves one row of each
  float* part_g;          // fp32
  float* part_b;          // fp32 (LayerNorm only)
  float* part_dres;       // fp32 or null: of dres (a bias gradient)
  float* part_dx;         // fp32 or null: of dx (a bias gradient)
  int rows, h, rms;
  int slice_rows;         // divides rows; 0: one slice of all rows
  int slice_blocks;       // workgroups (and partial rows) per slice; 0: norm_bwd_blocks(slice_rows)
  int join;               // 1: held back for the weight gradients' launch (see HeldTail)
};

// What goes into the launch of weight gradients besides their tiles: the first stages of the bias gradients, and in a small block
// the Norm1 backward that it ends with.  None of them reads what another writes, so they can be one launch (GemmArgs::tail): column sums
// that follow on the same stream, behind a Norm1 backward with `join` or without one (norm.rows 0), are held back (per thread) until
// the weight gradients of that stream are launched with `tail` set.
struct ColsumPartial { const void* g; long ld; int rows, n; float* part; };
constexpr int COLSUM_MAX_HELD = 2;
struct HeldTail {
  static constexpr int MAX_H = 2048;         // rows of four waves: the fewest that a workgroup of a product has
  NormBwdArgs norm;
  ColsumPartial sums[COLSUM_MAX_HELD];
  int nsums;
  hipStream_t stream;
  bool open;
};
inline thread_local HeldTail t_tail{};

// Workgroups of the backward, per slice of a launch over `slices` slices (where the caller's memory allows their number to be
// chosen; the single-kernel entry point's scratch holds norm_bwd_blocks): one per compute unit, more where a row has few
// waves, so that about eight waves have their loads in flight.  Each leaves a partial row per gradient vector, which costs
// traffic, so there are no more than that, and each has four rows or more (us, 256 / 512 / 768: 16384 x 2560, five waves, 69.8 / 72.5 /
// 76; 8192 x 5120, ten, 69.3 / 75.8 / 83.7; 2048 x 5120 23.4 / 29.0 / 34.8; 4096 x 2048, four, 18.9 / 18.9 / 19.9; 8192 x 1024, two, 25.8 / 20.7 / 18.2).
inline int norm_bwd_slice_blocks(int slices, int slice_rows, int h) {
  const int waves = (h / 8 + 63) / 64, fill = 256 * (waves > 4 ? 1 : 8 / waves) / slices, want = (slice_rows + 3) / 4;
  return fill < 1 ? 1 : want < fill ? want : fill;
}
// Whether a launch's rows outgrow the last-level cache (256 MB, shared with the products beside them): tensors of 32 MB and
// more.  Then what is read once (x, the other ranks' sum, the incoming gradients but the one just written) and what is written
// goes past the caches: backward 16384 x 2560 79.8 -> 69.8 us, 8192 x 4096 63.5 -> 53.6, 4096 x 5120 44.1 -> 39.6; forward with the residual
// sum 73.3 -> 64.2, 58.7 -> 52.5, 38.8 -> 35.1.  Smaller ones are read again while they are still there: a step of 2 x 200
// tokens of a 1024-wide block 126.5 us without and 129.6 with, 2048 tokens of 13B 664.7 and 673.6, 6018 of 2.7B 623.4 and 627.6.
// Between 2^24 and 2^25 values the two sides meet (steps and forwards, without / with: 2048-wide 8192 tokens 551 / 559 and 208 / 203,
// 14336 tokens 882 / 871 and 321 / 325; 4096-wide 4096 tokens 754 / 761, 6144 1061 / 1055; 2560-wide 8192 tokens 734 / 738 and 274 / 268).
inline bool norm_streams(long rows, int h) { return rows * h >= 1L << 24; }

int norm_bwd_blocks(int rows);              // 16 rows each until the block limit is reached
hipError_t norm_fwd_launch(const NormFwdArgs& a, hipStream_t st);
hipError_t norm_bwd_launch(const NormBwdArgs& a, hipStream_t st);
// out[n] (+)= sum over nparts rows of part[nparts][n], summed in index order
hipError_t colsum_finish_launch(const float* part, int nparts, int n, float* out, int accumulate, hipStream_t st);
// several such reductions in one launch; a job sums nouter groups (ostride floats apart) of nparts
// partial rows (stride floats apart), group by group
constexpr int COLSUM_MAX_JOBS = 8;
struct ColsumJob { const float* part; float* out; int nparts, n; long stride; int nouter; long ostride; };
struct ColsumJobs {
  ColsumJob job[COLSUM_MAX_JOBS];
  int join;      // 1: hold these jobs back until the next call (same stream), which continues them with the groups behind theirs
};
hipError_t colsum_finish_jobs_launch(const ColsumJobs& jobs, int njobs, int accumulate, hipStream_t st);
// part[COLSUM_PARTS][n] = partial column sums of the bf16 matrix g[rows][ld]
hipError_t colsum_partial_launch(const void* g, long ld, int rows, int n, float* part, hipStream_t st);
