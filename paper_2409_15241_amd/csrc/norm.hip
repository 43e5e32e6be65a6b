// LayerNorm / RMSNorm forward and backward with the surrounding residual traffic fused in
// (the "dropout, residual, LayerNorm" group of Sec. 4.1.1, dropout-free; RMSNorm per Sec. 5.4).
// HBM-bound: every access is a 16-byte chunk and a wave's 64 lanes cover 1 KiB contiguous bytes per
// instruction.  Statistics are fp32; wave reductions combined through LDS give the row sums.
#include "norm_body.h"
#include <type_traits>

namespace {

// y = Norm(x + add1 + add2 + vec) * gamma + beta; optionally writes the pre-norm sum (bf16) too.
// The statistics are taken from the bf16-rounded sum, i.e. from exactly what the backward re-reads.
// A workgroup of four waves owns one row, thread t the 16-byte chunks t, t+256, ... (at most 4: hidden <= 8192);
// every load of a phase is issued before the first is used (chunks past the row end read the last chunk instead
// of branching, and are masked out of the sums and stores); the two row sums cross the waves through LDS in wave
// order.  Under 96 registers a lane: such waves fit beside the two 192-register waves that a 256x256 product
// tile keeps on every SIMD.
template <int NC, bool RMS, bool ONCE>
__global__ __launch_bounds__(256, 5)
void norm_fwd_kernel(const NormFwdArgs p) {
  __shared__ float red[2][4];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int row = blockIdx.x;
  const int nch = p.h >> 3;
  const long ro = (long)row * p.h;
  const u32x4* x = reinterpret_cast<const u32x4*>(static_cast<const bf16_t*>(p.x) + ro);
  const u32x4* a1 = p.add1 ? reinterpret_cast<const u32x4*>(static_cast<const bf16_t*>(p.add1) + ro) : nullptr;
  const u32x4* a2 = p.add2 ? reinterpret_cast<const u32x4*>(static_cast<const bf16_t*>(p.add2) + ro) : nullptr;
  const u32x4* vec = reinterpret_cast<const u32x4*>(p.vec);
  const bool fused = a1 || a2 || vec;
  const u32x4 zero4 = {0u, 0u, 0u, 0u};

  int cc[NC];
  bool live[NC];
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    const int c = tid + 256 * i;
    live[i] = c < nch;
    cc[i] = live[i] ? c : nch - 1;
  }
  u32x4 xs[NC];
#pragma unroll
  for (int i = 0; i < NC; ++i) xs[i] = fused ? load_row<ONCE>(x + cc[i]) : x[cc[i]];
  if (fused) {
    u32x4 t1[NC], t2[NC], t3[NC];
#pragma unroll
    for (int i = 0; i < NC; ++i) t1[i] = a1 ? a1[cc[i]] : zero4;
#pragma unroll
    for (int i = 0; i < NC; ++i) t2[i] = a2 ? load_row<ONCE>(a2 + cc[i]) : zero4;
#pragma unroll
    for (int i = 0; i < NC; ++i) t3[i] = vec ? vec[cc[i]] : zero4;
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      float f[8], g[8];
      unpack8(xs[i], f);
      unpack8(t1[i], g);
#pragma unroll
      for (int e = 0; e < 8; ++e) f[e] += g[e];
      unpack8(t2[i], g);
#pragma unroll
      for (int e = 0; e < 8; ++e) f[e] += g[e];
      unpack8(t3[i], g);
#pragma unroll
      for (int e = 0; e < 8; ++e) f[e] += g[e];
      xs[i] = pack8(f);
    }
    if (p.xsum) {
      u32x4* o = reinterpret_cast<u32x4*>(static_cast<bf16_t*>(p.xsum) + ro);
#pragma unroll
      for (int i = 0; i < NC; ++i)
        if (live[i]) store_row<ONCE>(o + cc[i], xs[i]);
    }
  }
  const u32x4* gam = reinterpret_cast<const u32x4*>(p.gamma);
  const u32x4* bet = reinterpret_cast<const u32x4*>(p.beta);
  u32x4 gs[NC], bs[NC];
#pragma unroll
  for (int i = 0; i < NC; ++i) gs[i] = gam[cc[i]];
  if (bet) {
#pragma unroll
    for (int i = 0; i < NC; ++i) bs[i] = bet[cc[i]];
  }

  const float inv_h = 1.0f / (float)p.h;
  float mean = 0.0f;
  if (!RMS) {
    float s = 0.0f;
#pragma unroll
    for (int i = 0; i < NC; ++i) {
      float f[8]; unpack8(xs[i], f);
      float t = 0.0f;
#pragma unroll
      for (int e = 0; e < 8; ++e) t += f[e];
      s += live[i] ? t : 0.0f;
    }
    s = wave_sum(s);
    if (lane == 0) red[0][wave] = s;
    __syncthreads();
    mean = (((red[0][0] + red[0][1]) + red[0][2]) + red[0][3]) * inv_h;
  }
  float ss = 0.0f;
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    float f[8]; unpack8(xs[i], f);
    float t = 0.0f;
#pragma unroll
    for (int e = 0; e < 8; ++e) { const float d = f[e] - mean; t += d * d; }
    ss += live[i] ? t : 0.0f;
  }
  ss = wave_sum(ss);
  if (lane == 0) red[1][wave] = ss;
  __syncthreads();
  const float rstd = rsqrtf((((red[1][0] + red[1][1]) + red[1][2]) + red[1][3]) * inv_h + p.eps);
  if (tid == 0) {
    if (p.mean) p.mean[row] = mean;
    p.rstd[row] = rstd;
  }
  u32x4* y = reinterpret_cast<u32x4*>(static_cast<bf16_t*>(p.y) + ro);
#pragma unroll
  for (int i = 0; i < NC; ++i) {
    float f[8], g[8];
    unpack8(xs[i], f);
    unpack8(gs[i], g);
#pragma unroll
    for (int e = 0; e < 8; ++e) f[e] = (f[e] - mean) * rstd * g[e];
    if (bet) {
      unpack8(bs[i], g);
#pragma unroll
      for (int e = 0; e < 8; ++e) f[e] += g[e];
    }
    if (live[i]) store_row<ONCE>(y + cc[i], pack8(f));
  }
}

template <int NT, int R, bool RMS, bool SUMS, bool ONCE>
__global__ __launch_bounds__(NT)
void norm_bwd_kernel(const NormBwdArgs p) {
  __shared__ __align__(16) float smem[norm_bwd_lds<R>(NT / 64) / 4];
  norm_bwd_body<R, RMS, SUMS, ONCE>(p, blockIdx.x, gridDim.x, smem);
}

// out[col] (+)= sum_k part[k][col]: the second stage of every column reduction, for up to
// COLSUM_MAX_JOBS independent reductions in one launch (blockIdx.y = job).  A workgroup owns 32
// columns; its 8 row groups each sum every 8th partial row, then the 8 group sums are added in
// group order (a fixed summation tree: results do not depend on scheduling).
__global__ __launch_bounds__(256)
void colsum_finish_kernel(const ColsumJobs jobs, int accumulate) {
  __shared__ float red[8][32];
  const ColsumJob job = jobs.job[blockIdx.y];
  if ((int)blockIdx.x * 32 >= job.n) return;
  const int c = threadIdx.x & 31, kg = threadIdx.x >> 5;
  const int col = blockIdx.x * 32 + c;
  float s = 0.0f;
  if (col < job.n) {
    for (int g = 0; g < job.nouter; ++g) {
      const float* part = job.part + (long)g * job.ostride + col;
      for (int k = kg; k < job.nparts; k += 128) {       // 16 rows in flight (four: 13 us where there are 2048 rows of 2560, 10 so)
        float v[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) v[j] = k + 8 * j < job.nparts ? part[(long)(k + 8 * j) * job.stride] : 0.0f;
#pragma unroll
        for (int j = 0; j < 16; ++j) s += v[j];
      }
    }
  }
  red[kg][c] = s;
  __syncthreads();
  if (kg == 0 && col < job.n) {
    float t = red[0][c];
#pragma unroll
    for (int g = 1; g < 8; ++g) t += red[g][c];
    job.out[col] = accumulate ? job.out[col] + t : t;
  }
}

__global__ __launch_bounds__(256)
void colsum_partial_kernel(const bf16_t* __restrict__ g, long ld, int rows, int n, float* __restrict__ part) {
  __shared__ __align__(16) float smem[COLSUM_LDS / 4];
  colsum_partial_body(g, ld, rows, n, part, blockIdx.x, blockIdx.y, gridDim.y, threadIdx.x >> 6, smem);
}

template <bool RMS, bool ONCE>
hipError_t fwd_dispatch(const NormFwdArgs& a, hipStream_t st) {
  const int nq = ((a.h >> 3) + 255) / 256;               // 16-byte chunks per thread
  const dim3 grid(a.rows), block(256);
  if (nq <= 1) hipLaunchKernelGGL((norm_fwd_kernel<1, RMS, ONCE>), grid, block, 0, st, a);
  else if (nq <= 2) hipLaunchKernelGGL((norm_fwd_kernel<2, RMS, ONCE>), grid, block, 0, st, a);
  else if (nq <= 3) hipLaunchKernelGGL((norm_fwd_kernel<3, RMS, ONCE>), grid, block, 0, st, a);
  else hipLaunchKernelGGL((norm_fwd_kernel<4, RMS, ONCE>), grid, block, 0, st, a);
  return hipGetLastError();
}

template <bool RMS, bool SUMS, bool ONCE>
hipError_t bwd_dispatch(const NormBwdArgs& a, hipStream_t st) {
  const int nt = (((a.h >> 3) + 63) / 64) * 64;           // one thread per 16-byte chunk of a row
  const dim3 grid(a.slice_blocks * (a.rows / a.slice_rows)), block(nt);
  // two rows per iteration (four took 245 registers and left one workgroup per compute unit), one where the block has 16 waves
  if (nt <= 256) hipLaunchKernelGGL((norm_bwd_kernel<256, 2, RMS, SUMS, ONCE>), grid, block, 0, st, a);
  else if (nt <= 512) hipLaunchKernelGGL((norm_bwd_kernel<512, 2, RMS, SUMS, ONCE>), grid, block, 0, st, a);
  else if (nt <= 768) hipLaunchKernelGGL((norm_bwd_kernel<768, 2, RMS, SUMS, ONCE>), grid, block, 0, st, a);
  else hipLaunchKernelGGL((norm_bwd_kernel<1024, 1, RMS, SUMS, ONCE>), grid, block, 0, st, a);
  return hipGetLastError();
}

}  // namespace

int norm_bwd_blocks(int rows) {
  const int want = (rows + NORM_BWD_ROWS - 1) / NORM_BWD_ROWS;
  return want < NORM_BWD_MAX_BLOCKS ? want : NORM_BWD_MAX_BLOCKS;
}

hipError_t norm_fwd_launch(const NormFwdArgs& a, hipStream_t st) {
  if (norm_streams(a.rows, a.h)) return a.rms ? fwd_dispatch<true, true>(a, st) : fwd_dispatch<false, true>(a, st);
  return a.rms ? fwd_dispatch<true, false>(a, st) : fwd_dispatch<false, false>(a, st);
}

hipError_t norm_bwd_launch(const NormBwdArgs& a0, hipStream_t st) {
  NormBwdArgs a = a0;
  if (a.slice_rows <= 0) a.slice_rows = a.rows;
  if (a.slice_blocks <= 0) a.slice_blocks = norm_bwd_blocks(a.slice_rows);
  if (a.rows % a.slice_rows) return hipErrorInvalidValue;
  if (a.join) {
    t_tail = HeldTail{a, {}, 0, st, true};
    return hipSuccess;
  }
  const bool sums = a.part_dres && a.part_dx && a.dres;
  auto form = [&](auto once) {
    constexpr bool ONCE = decltype(once)::value;
    if (a.rms) return sums ? bwd_dispatch<true, true, ONCE>(a, st) : bwd_dispatch<true, false, ONCE>(a, st);
    return sums ? bwd_dispatch<false, true, ONCE>(a, st) : bwd_dispatch<false, false, ONCE>(a, st);
  };
  return norm_streams(a.rows, a.h) ? form(std::true_type{}) : form(std::false_type{});
}

hipError_t colsum_finish_launch(const float* part, int nparts, int n, float* out, int accumulate, hipStream_t st) {
  ColsumJobs jobs{};
  jobs.job[0] = {part, out, nparts, n, (long)n, 1, 0};
  return colsum_finish_jobs_launch(jobs, 1, accumulate, st);
}

namespace {
// jobs held back for the next call (ColsumJobs::join)
thread_local ColsumJobs t_held;
thread_local int t_nheld = 0, t_accumulate = 0;
}  // namespace

hipError_t colsum_finish_jobs_launch(const ColsumJobs& jobs0, int njobs, int accumulate, hipStream_t st) {
  if (njobs <= 0) return hipSuccess;
  if (njobs > COLSUM_MAX_JOBS) return hipErrorInvalidValue;
  ColsumJobs jobs = jobs0;
  if (t_nheld) {
    ColsumJobs held = t_held;
    const int nheld = t_nheld;
    t_nheld = 0;
    for (int k = 0; k < njobs; ++k) {           // every job must lengthen a held one
      int h = 0;
      while (h < nheld && held.job[h].out != jobs.job[k].out) ++h;
      if (h == nheld || !accumulate) return hipErrorInvalidValue;
      ColsumJob& j = held.job[h];
      const ColsumJob& more = jobs.job[k];
      if (j.n != more.n || j.nparts != more.nparts || j.stride != more.stride || j.ostride != more.ostride ||
          j.part + j.nouter * j.ostride != more.part) return hipErrorInvalidValue;
      j.nouter += more.nouter;
    }
    jobs = held; njobs = nheld; accumulate = t_accumulate;
  }
  if (jobs0.join) {
    t_held = jobs; t_nheld = njobs; t_accumulate = accumulate;
    return hipSuccess;
  }
  int widest = 0;
  for (int k = 0; k < njobs; ++k) widest = jobs.job[k].n > widest ? jobs.job[k].n : widest;
  hipLaunchKernelGGL(colsum_finish_kernel, dim3((widest + 31) / 32, njobs), dim3(256), 0, st, jobs, accumulate);
  return hipGetLastError();
}

hipError_t colsum_partial_launch(const void* g, long ld, int rows, int n, float* part, hipStream_t st) {
  if (t_tail.open && t_tail.stream == st && t_tail.nsums < COLSUM_MAX_HELD) {
    t_tail.sums[t_tail.nsums++] = {g, ld, rows, n, part};
    return hipSuccess;
  }
  hipLaunchKernelGGL(colsum_partial_kernel, dim3((n / 8 + 63) / 64, COLSUM_PARTS), dim3(256), 0, st,
                     static_cast<const bf16_t*>(g), ld, rows, n, part);
  return hipGetLastError();
}
