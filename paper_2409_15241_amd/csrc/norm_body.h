// Device code of the norm backward and of the column sums' first stage: as kernels of their own (norm.hip) and as further
// workgroups of the launch that forms a small block's weight gradients (gemm.hip).
#pragma once
#include "common.h"
#include "norm.h"

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

// dx = dres + NormBwd(ga + gb); per-workgroup partial sums of d gamma / d beta.
// The launch's workgroups sweep the rows side by side, R rows each at a time; thread t owns the 8 columns of 16-byte chunk t in
// every row, so its share of the column sums (d gamma, d beta) is 16 registers and every load of an iteration (R rows x up
// to 4 tensors) is in flight at once.  Side by side the memory sees one front per tensor: with a range of rows to each workgroup
// 16384 x 2560 took 88.1 us and 80.4 so (512 and 256 workgroups), 8192 x 4096 67.7 and 63.5, 8192 x 5120 95.8 and 88.0.  The two
// row sums cross the waves through LDS: wave sums in a double-buffered table, one barrier per
// iteration, added in wave order (fixed summation order).
// `block` of `blocks` workgroups; smem: norm_bwd_lds<R>(waves) bytes.  Waves behind the row's end only take part in the barriers.
template <int R> constexpr int norm_bwd_rw() { return 2 * R < 4 ? 4 : 2 * R; }      // row sums per wave and iteration, padded to whole 16-byte reads
template <int R> constexpr int norm_bwd_lds(int waves) { return 2 * waves * norm_bwd_rw<R>() * 4; }
template <int R, bool RMS, bool SUMS, bool ONCE>
DEV void norm_bwd_body(const NormBwdArgs& p, int block, int blocks, float* smem) {
  constexpr int RW = norm_bwd_rw<R>();
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int nch = p.h >> 3, nw = (nch + 63) >> 6;
  auto red = [&](int buf, int w) { return smem + (buf * nw + w) * RW; };
  const bool live = tid < nch;
  const float inv_h = 1.0f / (float)p.h;
  const u32x4 zero4 = {0u, 0u, 0u, 0u};

  float gm[8];
  unpack8(live ? reinterpret_cast<const u32x4*>(p.gamma)[tid] : zero4, gm);
  float dg[8], db[8], sres[8], sdx[8];     // sres / sdx: column sums of dres and of dx (SUMS only)
#pragma unroll
  for (int e = 0; e < 8; ++e) { dg[e] = 0.0f; db[e] = 0.0f; sres[e] = 0.0f; sdx[e] = 0.0f; }

  const int r1 = p.rows, step = blocks * R;
  const long part_at = (long)block * p.h + tid * 8;
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
  load_rows(block * R, cur);
  int buf = 0;
  for (int rb = block * R; rb < r1; rb += step, buf ^= 1) {
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
    if (lane == 0 && wave < nw) {
#pragma unroll
      for (int k = 0; k < RW; ++k) red(buf, wave)[k] = k < 2 * R ? sums[k] : 0.0f;
    }
    __syncthreads();
    float tot[RW];
#pragma unroll
    for (int k = 0; k < RW; ++k) tot[k] = 0.0f;
    for (int w = 0; w < nw; ++w) {
#pragma unroll
      for (int k4 = 0; k4 < RW; k4 += 4) {
        const f32x4 t = *reinterpret_cast<const f32x4*>(red(buf, w) + k4);
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

// part[range][col] = sum over one of `ranges` row ranges of g[row][col] (bf16 in, fp32 out).  HBM-bound: a workgroup owns
// 512 columns, its four waves take every fourth row of the range with eight 1-KiB loads in flight each, and the wave sums
// are added in wave order through LDS.  (One wave per workgroup and four loads in flight read 16384 x 1280 at 1.4 TB/s.)
// `wave` of the four; smem: COLSUM_LDS bytes.  All threads of the workgroup take part in the one barrier.
constexpr int COLSUM_LDS = 3 * 512 * 4;
DEV void colsum_partial_body(const bf16_t* __restrict__ g, long ld, int rows, int n, float* __restrict__ part, int column_block, int range,
                             int ranges, int wave, float* smem) {
  auto red = [&](int w) { return smem + w * 512; };
  const int lane = threadIdx.x & 63;
  const int chunk = column_block * 64 + lane;             // 8 columns
  const bool live = chunk * 8 < n;
  const bf16_t* at = g + (live ? chunk : 0) * 8;
  const int per = (rows + ranges - 1) / ranges;
  const int r0 = range * per, r1 = min(rows, r0 + per);
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
    for (int e = 0; e < 8; e += 4) *reinterpret_cast<f32x4*>(red(wave - 1) + lane * 8 + e) = f32x4{acc[e], acc[e + 1], acc[e + 2], acc[e + 3]};
  }
  __syncthreads();
  if (wave || !live) return;
#pragma unroll
  for (int w = 0; w < 3; ++w)
#pragma unroll
    for (int e = 0; e < 8; ++e) acc[e] += red(w)[lane * 8 + e];
  f32x4* o = reinterpret_cast<f32x4*>(part + (long)range * n + chunk * 8);
  o[0] = f32x4{acc[0], acc[1], acc[2], acc[3]};
  o[1] = f32x4{acc[4], acc[5], acc[6], acc[7]};
}
