// LayerNorm / RMSNorm forward and backward with the surrounding residual traffic fused in
// (the "dropout, residual, LayerNorm" group of Sec. 4.1.1, dropout-free; RMSNorm per Sec. 5.4).
// HBM-bound: every access is a 16-byte chunk and a wave's 64 lanes cover 1 KiB contiguous bytes per
// instruction.  Statistics are fp32; wave reductions combined through LDS give the row sums.
#include "norm.h"
#include "common.h"
#include <type_traits>

namespace {

DEV void unpack8(const u32x4 v, float* f) {
  f[0] = bf16_lo(v[0]); f[1] = bf16_hi(v[0]); f[2] = bf16_lo(v[1]); f[3] = bf16_hi(v[1]);
  f[4] = bf16_lo(v[2]); f[5] = bf16_hi(v[2]); f[6] = bf16_lo(v[3]); f[7] = bf16_hi(v[3]);
}
// ONCE: rows that nobody reads again soon go past the caches (see norm_streams)
template <bool ONCE>
DEV u32x4 load_row(const u32x4* p) {
  if constexpr (ONCE) return __builtin_nontemporal_load(p); else return *p;
}
template <bool ONCE>
DEV void store_row(u32x4* p, const u32x4 v) {
  if constexpr (ONCE) __builtin_nontemporal_store(v, p); else *p = v;
}
DEV u32x4 pack8(const float* f) {
  u32x4 v = {pack_bf16(f[0], f[1]), pack_bf16(f[2], f[3]), pack_bf16(f[4], f[5]), pack_bf16(f[6], f[7])};
  return v;
}

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

// dx = dres + NormBwd(ga + gb); per-workgroup partial sums of d gamma / d beta.
// The launch's workgroups sweep the rows side by side, R rows each at a time; thread t owns the 8 columns of 16-byte chunk t in
// every row, so its share of the column sums (d gamma, d beta) is 16 registers and every load of an iteration (R rows x up
// to 4 tensors) is in flight at once.  Side by side the memory sees one front per tensor: with a range of rows to each workgroup
// 16384 x 2560 took 88.1 us and 80.4 so (512 and 256 workgroups), 8192 x 4096 67.7 and 63.5, 8192 x 5120 95.8 and 88.0.  The two
// row sums cross the waves through LDS: wave sums in a double-buffered table, one barrier per
// iteration, added in wave order (fixed summation order).
template <int NT, int R, bool RMS, bool SUMS, bool ONCE>
__global__ __launch_bounds__(NT)
void norm_bwd_kernel(const NormBwdArgs p) {
  constexpr int NW = NT / 64;
  constexpr int RW = 2 * R < 4 ? 4 : 2 * R;     // row sums per wave and iteration, padded to whole 16-byte reads
  __shared__ __align__(16) float red[2][NW][RW];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int nw = blockDim.x >> 6;
  const int nch = p.h >> 3;
  const bool live = tid < nch;
  const float inv_h = 1.0f / (float)p.h;
  const u32x4 zero4 = {0u, 0u, 0u, 0u};

  float gm[8];
  unpack8(live ? reinterpret_cast<const u32x4*>(p.gamma)[tid] : zero4, gm);
  float dg[8], db[8], sres[8], sdx[8];     // sres / sdx: column sums of dres and of dx (SUMS only)
#pragma unroll
  for (int e = 0; e < 8; ++e) { dg[e] = 0.0f; db[e] = 0.0f; sres[e] = 0.0f; sdx[e] = 0.0f; }

  const int r1 = p.rows, step = gridDim.x * R;
  const long part_at = (long)blockIdx.x * p.h + tid * 8;
  // the rows of iteration k+1 are requested before iteration k is worked on, so the memory pipeline stays
  // busy across the barrier and the arithmetic of an iteration
  struct Rows { u32x4 xs[R], gs[R], bs[R], ds[R]; float mean[R], rstd[R]; };
  auto load_rows = [&](int rb, Rows& w) {
#pragma unroll
    for (int j = 0; j < R; ++j) {
      const int row = rb + j;
      const bool ok = live && row < r1;
      const long at = (long)row * p.h + tid * 8;
      w.xs[j] = ok ? load_row<ONCE>(reinterpret_cast<const u32x4*>(static_cast<const bf16_t*>(p.x) + at)) : zero4;
      w.gs[j] = ok ? *reinterpret_cast<const u32x4*>(static_cast<const bf16_t*>(p.ga) + at) : zero4;
      w.bs[j] = (ok && p.gb) ? load_row<ONCE>(reinterpret_cast<const u32x4*>(static_cast<const bf16_t*>(p.gb) + at)) : zero4;
      w.ds[j] = (ok && p.dres) ? load_row<ONCE>(reinterpret_cast<const u32x4*>(static_cast<const bf16_t*>(p.dres) + at)) : zero4;
      w.mean[j] = (!RMS && row < r1) ? p.mean[row] : 0.0f;
      w.rstd[j] = row < r1 ? p.rstd[row] : 0.0f;
    }
  };
  Rows cur, nxt;
  load_rows(blockIdx.x * R, cur);
  int buf = 0;
  for (int rb = blockIdx.x * R; rb < r1; rb += step, buf ^= 1) {
    load_rows(rb + step, nxt);                     // rows past r1 load nothing
    const u32x4 (&xs)[R] = cur.xs;
    const u32x4 (&gs)[R] = cur.gs;
    const u32x4 (&bs)[R] = cur.bs;
    const u32x4 (&ds)[R] = cur.ds;
    const float (&mean)[R] = cur.mean;
    const float (&rstd)[R] = cur.rstd;
    float sums[2 * R];
#pragma unroll
    for (int j = 0; j < R; ++j) {
      float xv[8], gv[8], bv[8];
      unpack8(xs[j], xv); unpack8(gs[j], gv); unpack8(bs[j], bv);
      float s1 = 0.0f, s2 = 0.0f;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        gv[e] += bv[e];
        const float xh = (xv[e] - mean[j]) * rstd[j];
        const float dxh = gv[e] * gm[e];
        s1 += dxh;
        s2 += dxh * xh;
        dg[e] += gv[e] * xh;
        if (!RMS) db[e] += gv[e];
      }
      sums[2 * j] = RMS ? 0.0f : wave_sum(s1);
      sums[2 * j + 1] = wave_sum(s2);
    }
    if (lane == 0) {
#pragma unroll
      for (int k = 0; k < RW; ++k) red[buf][wave][k] = k < 2 * R ? sums[k] : 0.0f;
    }
    __syncthreads();
    float tot[RW];
#pragma unroll
    for (int k = 0; k < RW; ++k) tot[k] = 0.0f;
    for (int w = 0; w < nw; ++w) {
#pragma unroll
      for (int k4 = 0; k4 < RW; k4 += 4) {
        const f32x4 t = *reinterpret_cast<const f32x4*>(&red[buf][w][k4]);
#pragma unroll
        for (int e = 0; e < 4; ++e) tot[k4 + e] += t[e];
      }
    }
#pragma unroll
    for (int j = 0; j < R; ++j) {
      const int row = rb + j;
      if (live && row < r1) {
        const float c1 = tot[2 * j] * inv_h, c2 = tot[2 * j + 1] * inv_h;
        float o[8], rv[8], xv[8], gv[8], bv[8];     // the incoming gradient is unpacked again rather than kept
        unpack8(ds[j], rv); unpack8(xs[j], xv); unpack8(gs[j], gv); unpack8(bs[j], bv);
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          o[e] = rstd[j] * ((gv[e] + bv[e]) * gm[e] - c1 - (xv[e] - mean[j]) * rstd[j] * c2) + rv[e];
          if (SUMS) { sres[e] += rv[e]; sdx[e] += o[e]; }
        }
        store_row<ONCE>(reinterpret_cast<u32x4*>(static_cast<bf16_t*>(p.dx) + (long)row * p.h + tid * 8), pack8(o));
      }
    }
    cur = nxt;
  }
  if (live) {
    f32x4* pg = reinterpret_cast<f32x4*>(p.part_g + part_at);
    pg[0] = f32x4{dg[0], dg[1], dg[2], dg[3]};
    pg[1] = f32x4{dg[4], dg[5], dg[6], dg[7]};
    if (!RMS) {
      f32x4* pb = reinterpret_cast<f32x4*>(p.part_b + part_at);
      pb[0] = f32x4{db[0], db[1], db[2], db[3]};
      pb[1] = f32x4{db[4], db[5], db[6], db[7]};
    }
    if (SUMS) {
      f32x4* pr = reinterpret_cast<f32x4*>(p.part_dres + part_at);
      pr[0] = f32x4{sres[0], sres[1], sres[2], sres[3]};
      pr[1] = f32x4{sres[4], sres[5], sres[6], sres[7]};
      f32x4* px = reinterpret_cast<f32x4*>(p.part_dx + part_at);
      px[0] = f32x4{sdx[0], sdx[1], sdx[2], sdx[3]};
      px[1] = f32x4{sdx[4], sdx[5], sdx[6], sdx[7]};
    }
  }
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

// part[blockIdx.y][col] = sum over this block's row range of g[row][col] (bf16 in, fp32 out).  HBM-bound: a workgroup owns
// 512 columns, its four waves take every fourth row of the range with eight 1-KiB loads in flight each, and the wave sums
// are added in wave order through LDS.  (One wave per workgroup and four loads in flight read 16384 x 1280 at 1.4 TB/s.)
__global__ __launch_bounds__(256)
void colsum_partial_kernel(const bf16_t* __restrict__ g, long ld, int rows, int n, float* __restrict__ part) {
  __shared__ __align__(16) float red[3][512];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int chunk = blockIdx.x * 64 + lane;             // 8 columns
  const bool live = chunk * 8 < n;
  const bf16_t* at = g + (live ? chunk : 0) * 8;
  const int per = (rows + gridDim.y - 1) / gridDim.y;
  const int r0 = blockIdx.y * per, r1 = min(rows, r0 + per);
  float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
  int r = r0 + wave;
  for (; r + 28 < r1; r += 32) {
    u32x4 v[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) v[k] = *reinterpret_cast<const u32x4*>(at + (long)(r + 4 * k) * ld);
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      float f[8];
      unpack8(v[k], f);
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] += f[e];
    }
  }
  for (; r < r1; r += 4) {
    float f[8];
    unpack8(*reinterpret_cast<const u32x4*>(at + (long)r * ld), f);
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] += f[e];
  }
  if (wave) {
#pragma unroll
    for (int e = 0; e < 8; e += 4) *reinterpret_cast<f32x4*>(&red[wave - 1][lane * 8 + e]) = f32x4{acc[e], acc[e + 1], acc[e + 2], acc[e + 3]};
  }
  __syncthreads();
  if (wave || !live) return;
#pragma unroll
  for (int w = 0; w < 3; ++w)
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] += red[w][lane * 8 + e];
  f32x4* o = reinterpret_cast<f32x4*>(part + (long)blockIdx.y * n + chunk * 8);
  o[0] = f32x4{acc[0], acc[1], acc[2], acc[3]};
  o[1] = f32x4{acc[4], acc[5], acc[6], acc[7]};
}

// Whether a launch's rows outgrow the last-level cache (256 MB, shared with the products beside them): tensors of 32 MB and
// more.  Then what is read once (x, the other ranks' sum, the incoming gradients but the one just written) and what is written
// goes past the caches: backward 16384 x 2560 79.8 -> 69.8 us, 8192 x 4096 63.5 -> 53.6, 4096 x 5120 44.1 -> 39.6; forward with the residual
// sum 73.3 -> 64.2, 58.7 -> 52.5, 38.8 -> 35.1.  Smaller ones are read again while they are still there: a step of 2 x 200
// tokens of a 1024-wide block 126.5 us without and 129.6 with, 2048 tokens of 13B 664.7 and 673.6, 6018 of 2.7B 623.4 and 627.6.
bool norm_streams(long rows, int h) { return rows * h >= 1L << 24; }

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
  hipLaunchKernelGGL(colsum_partial_kernel, dim3((n / 8 + 63) / 64, COLSUM_PARTS), dim3(256), 0, st,
                     static_cast<const bf16_t*>(g), ld, rows, n, part);
  return hipGetLastError();
}
