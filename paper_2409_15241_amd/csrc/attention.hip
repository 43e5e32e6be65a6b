// Causal flash-style attention for one head shard on gfx950 MFMA (Eq. 2, first case:
// softmax(Q K^T / sqrt(d_k)) V; kept as one fused kernel because the first weight group is never
// sliced, Sec. 3.1), forward and backward.
//
// All products are computed transposed so that the query (forward, dQ pass) or key (dK/dV pass)
// index of an MFMA accumulator is the LANE and the other index lives in the lane's 16 registers:
//   S^T[kv, q] = K Q^T          row statistics of a query are then a reduction over one lane's
//   O^T[d, q]  = V^T P^T        registers plus one exchange between the two lane halves, and the
// probabilities never leave registers: an accumulator converted to bf16 is directly the second
// operand of the next product, provided the first operand's contraction index is read in the
// accumulator's row order (the transposing LDS reads below take their rows in that order).
// Operand tiles travel HBM/L2 -> LDS with buffer_load ... lds, double buffered; see lds_dma.h.
//
// Backward is two passes without atomics (run-to-run identical results):
//   dQ pass, one workgroup per 128 queries: recompute P^T from the saved log-sum-exp,
//     dP^T = V dO^T, dS^T = P^T (dP^T - D), dQ^T += K^T dS^T.
//   dK/dV pass, one workgroup per 128 keys: P = exp(S - lse), dV^T += dO^T P, dP = dO V^T,
//     dS = P (dP - D), dK^T += Q^T dS.
// D[q] = sum_d dO[q,d] O[q,d] comes from a small pre-pass.
#include "attention.h"
#include "host_once.h"
#include "lds_dma.h"
#include <type_traits>

namespace {

// 2^x as the bare hardware instruction: the arguments here are differences to a running maximum or to the
// log-sum-exp (at most about 0; -inf for masked scores gives 0), where results below 2^-126 may flush to zero,
// so the range fix-up that the library's exp2f wraps around it (a compare, two selects and an ldexp per value)
// is dead weight on the vector ALUs that bound these kernels.
DEV float exp2_raw(float x) { return __builtin_amdgcn_exp2f(x); }
constexpr float LOG2E = 1.4426950408889634f;
constexpr float LN2 = 0.6931471805599453f;

template <int D>
struct Dims {
  static constexpr int DT = (D + 31) / 32;             // 32-row d tiles of a transposed (d x position) product
  static constexpr int KSTEPS = D / 16;               // MFMA steps of a contraction over d
};

// B-operand fragments straight from HBM: lane (pos = row0 + lane%32, half) takes 8 consecutive d.
template <int D>
DEV void load_row_frags(const bf16_t* __restrict__ base, long ld, int pos, int seq, int fh,
                        bf16x8 (&f)[Dims<D>::KSTEPS]) {
#pragma unroll
  for (int ks = 0; ks < Dims<D>::KSTEPS; ++ks) {
    u32x4 v = {0u, 0u, 0u, 0u};
    if (pos < seq) v = *reinterpret_cast<const u32x4*>(base + (long)pos * ld + ks * 16 + fh * 8);
    f[ks] = __builtin_bit_cast(bf16x8, v);
  }
}

// accumulator register v of the lane half fh holds tile row 8 (v/4) + 4 fh + v%4
DEV int acc_row(int v, int fh) { return 8 * (v >> 2) + 4 * fh + (v & 3); }

// store out^T[d, pos] (one lane = one position) as bf16 rows of a [pos][..] matrix, scaled
template <int D>
DEV void store_transposed(const f32x16 (&o)[Dims<D>::DT], float scale, bf16_t* __restrict__ row_ptr, int fh) {
#pragma unroll
  for (int dt = 0; dt < Dims<D>::DT; ++dt)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int dd = 32 * dt + 8 * g + 4 * fh;
      if (dd < D) {
        u32x2 w = {pack_bf16(o[dt][4 * g] * scale, o[dt][4 * g + 1] * scale),
                   pack_bf16(o[dt][4 * g + 2] * scale, o[dt][4 * g + 3] * scale)};
        *reinterpret_cast<u32x2*>(row_ptr + dd) = w;
      }
    }
}

// The rotary embedding's transpose on out^T[d, pos]: the gradient with respect to a rotated q or k, taken back to
// the vector before the rotation.  The pair (i, i + D/2) of a position sits in one lane (accumulator rows 32 dt + 8 g
// + 4 fh + e: adding D/2 = 32, 40 or 64 changes dt and g only), so nothing crosses lanes.
template <int D>
DEV void rope_back(f32x16 (&o)[Dims<D>::DT], int pos, int fh, float log2_base) {
  constexpr int H = D / 2;
  const float fpos = (float)pos;
#pragma unroll
  for (int dt = 0; dt < Dims<D>::DT; ++dt)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      const int dd0 = 32 * dt + 8 * g;               // this lane's rows of the group: dd0 + 4 fh + e
      if (dd0 < H) {
        const int dt2 = (dd0 + H) / 32, g2 = ((dd0 + H) % 32) / 8;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          float sn, cs;
          rope_sincos(fpos, rope_freq(dd0 + 4 * fh + e, D, log2_base), &sn, &cs);
          const float lo = o[dt][4 * g + e], hi = o[dt2][4 * g2 + e];
          o[dt][4 * g + e] = lo * cs + hi * sn;
          o[dt2][4 * g2 + e] = hi * cs - lo * sn;
        }
      }
    }
}

// compile-time loop: f(std::integral_constant<int, I>) for I in [0, N)
template <int I, int N, class F>
DEV void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<I + 1, N>(f);
  }
}

// Work order.  Workgroups differ in length by the causal mask (2 to 2 s/64 tiles), and the hardware deals
// consecutive workgroup ids round-robin over the 8 XCDs: with a plain (block, head, batch) grid the workgroups
// whose block index is a multiple of 8 (the longest of every head) all land on one XCD, which then carries
// 2.4 times the work of the last one.  So the launch is a 1-D grid and the work items are ranked instead: rank
// = (position of the item inside its (batch, head) group, longest first) * groups + group, dealt over the XCDs
// in snake order (0..7, 7..0, ...): every XCD gets the same mix, longest items first.  Returns the item's
// position inside its group and the group, or false for the padding workgroups of the last round.
DEV bool ranked_item(int per_group, int groups, int& pos, int& group) {
  const int id = __builtin_amdgcn_readfirstlane(blockIdx.x);
  const int xcd = id & 7, round = id >> 3;
  const int rank = round * 8 + ((round & 1) ? 7 - xcd : xcd);
  if (rank >= per_group * groups) return false;
  pos = rank / groups;
  group = rank % groups;
  return true;
}
inline int ranked_grid(int per_group, int groups) { return ((per_group * groups + 7) / 8) * 8; }

// ------------------------------------------------------------------------------------- D = rowsum(dO * O)
// One thread per (row, head), all its loads in flight at once; a workgroup of one wave, so that few rows still spread over
// the chip.  The sum runs along d as it always has: for a sequence of one position it equals the product that it is
// subtracted from bit for bit.
template <int D>
__global__ __launch_bounds__(64)
void attn_dot_kernel(const bf16_t* __restrict__ o, const bf16_t* __restrict__ dO, long ld, int rows, int seq,
                     int heads, float* __restrict__ dot) {
  const int i = blockIdx.x * 64 + threadIdx.x;
  if (i >= rows * heads) return;
  const int row = i / heads, hh = i % heads;
  const u32x4* a = reinterpret_cast<const u32x4*>(o + (long)row * ld + hh * D);
  const u32x4* b = reinterpret_cast<const u32x4*>(dO + (long)row * ld + hh * D);
  u32x4 x[D / 8], y[D / 8];
#pragma unroll
  for (int c = 0; c < D / 8; ++c) { x[c] = a[c]; y[c] = b[c]; }
  float acc = 0.0f;
#pragma unroll
  for (int c = 0; c < D / 8; ++c)
#pragma unroll
    for (int e = 0; e < 4; ++e) acc += bf16_lo(x[c][e]) * bf16_lo(y[c][e]) + bf16_hi(x[c][e]) * bf16_hi(y[c][e]);
  dot[((long)(row / seq) * heads + hh) * seq + row % seq] = acc;
}

// ------------------------------------------------------------------------------------- backward tiles
// Row-major LDS tile [64 positions][128 d] (16 KiB) filled by buffer_load ... lds, serving BOTH fragment
// kinds of one operand: the plain fragment (row = position, 8 consecutive d: ds_read_b128) and the
// transposed fragment (row = d, contraction over positions in accumulator-row order: two
// ds_read_b64_tr_b16).  16-byte chunk c of row r lives at r*256 + ((c ^ rm_swz(r)) << 4): the 16 rows of a
// plain read hit 16 distinct chunk positions, and the 4 rows x 2 column groups of a transposing
// read hit 8 distinct 32-byte pairs.
DEV int rm_swz(int r) { return ((r & 3) << 2) | ((r >> 2) & 3); }

struct RmLoader {            // 4 waves x 4 one-KiB pieces (4 rows each)
  uint32_t base[4];
  DEV void init(int ld, int d_valid, int wave, int lane) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int row = 4 * (wave * 4 + i) + (lane >> 4);
      const int d = ((lane & 15) ^ rm_swz(row)) * 8;
      base[i] = d < d_valid ? (uint32_t)(row * ld + d) * 2u : BUF_OOB;
    }
  }
  DEV void issue_one(int i, buf_rsrc rs, uint8_t* tile, uint32_t row_byte_off, int wave) const {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, LDS_PTR(tile + (wave * 4 + i) * 1024), 16, base[i] + row_byte_off, 0, 0, 0);
  }
  DEV void issue(buf_rsrc rs, uint8_t* tile, uint32_t row_byte_off, int wave) const {
#pragma unroll
    for (int i = 0; i < 4; ++i) issue_one(i, rs, tile, row_byte_off, wave);
  }
};
// per-lane byte offset of the plain fragment (row lane%32, chunk lane/32) at contraction step 0; step ks
// is reached by XOR (ks << 5), the second 32-row group by + 8192
DEV uint32_t rm_plain_off(int lane) {
  const int fr = lane & 31, fh = lane >> 5;
  return (uint32_t)(fr * 256 + ((fh ^ rm_swz(fr)) << 4));
}
// per-lane byte offset of the first transposing read of the transposed fragment (d tile 0); d tile dt and
// the second read are reached by XOR ((4 dt) ^ (2 second)) << 4; + 4096 u + 8192 sub + 2048 second
DEV uint32_t rm_trans_off(int lane) {
  const int sl = lane & 15, nh = (lane >> 4) & 1, fh = lane >> 5;
  const int posl = 4 * fh + (sl >> 2);
  const int h = (2 * nh + ((sl & 3) >> 1)) ^ rm_swz(posl);
  return (uint32_t)(posl * 256 + (h << 4) + 8 * (sl & 1));
}

// Both row products of 32 tile positions: accA += TileA[32 t + lane%32, d] * fa[d, lane] and accB likewise, over all d, in
// batches of a few steps with the next batch's reads in flight; the two chains of MFMAs alternate.  off = rm_plain_off(lane).
template <int D, int T>
DEV void rm_mma_rows(uint32_t tile_a, uint32_t tile_b, uint32_t off, const bf16x8 (&fa)[Dims<D>::KSTEPS], const bf16x8 (&fb)[Dims<D>::KSTEPS],
                     f32x16& acc_a, f32x16& acc_b) {
  using X = Dims<D>;
  constexpr int BS = D == 128 ? 4 : 2, NB = (X::KSTEPS + BS - 1) / BS;
  u32x4 fr[2][BS][2];
  auto read_batch = [&](auto bb) {
    constexpr int B = decltype(bb)::value;
    static_for<0, BS>([&](auto kk) {
      constexpr int KS = B * BS + decltype(kk)::value;
      if constexpr (KS < X::KSTEPS) {
        fr[B & 1][decltype(kk)::value][0] = ds_read_b128_at<T * 8192>(tile_a + (off ^ (KS << 5)));
        fr[B & 1][decltype(kk)::value][1] = ds_read_b128_at<T * 8192>(tile_b + (off ^ (KS << 5)));
      }
    });
  };
  read_batch(std::integral_constant<int, 0>{});
  static_for<0, NB>([&](auto bb) {
    constexpr int B = decltype(bb)::value;
    constexpr int LEFT = X::KSTEPS - BS * (B + 1);
    constexpr int NEXT = (B + 1 < NB) ? (LEFT < BS ? LEFT : BS) * 2 : 0;
    if constexpr (B + 1 < NB) read_batch(std::integral_constant<int, B + 1>{});
    lds_wait<NEXT>();
    static_for<0, BS>([&](auto kk) {
      constexpr int K = decltype(kk)::value, KS = B * BS + K;
      if constexpr (KS < X::KSTEPS) {
        tie(fr[B & 1][K][0]);
        tie(fr[B & 1][K][1]);
        acc_a = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, fr[B & 1][K][0]), fa[KS], acc_a, 0, 0, 0);
        acc_b = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, fr[B & 1][K][1]), fb[KS], acc_b, 0, 0, 0);
      }
    });
  });
}

// States that the running sums sit in the accumulation registers at this point.  Placed at the top of a pass's
// loop it keeps them there across the back edge; without it the register allocator carried them in vector registers at
// the loop head and copied them to the accumulation registers and back around every tile.
template <int N>
DEV void pin_acc(f32x16 (&acc)[N]) {
#pragma unroll
  for (int i = 0; i < N; ++i) asm volatile("" : "+a"(acc[i]));
}

// 16 accumulator values (32 tile positions), rounded to bf16 as the second operand of rm_mma_cols
DEV void pack_acc(const f32x16& vals, bf16x8 (&pf)[2]) {
#pragma unroll
  for (int u = 0; u < 2; ++u) {
    const u32x4 w = {pack_bf16(vals[8 * u + 0], vals[8 * u + 1]), pack_bf16(vals[8 * u + 2], vals[8 * u + 3]),
                     pack_bf16(vals[8 * u + 4], vals[8 * u + 5]), pack_bf16(vals[8 * u + 6], vals[8 * u + 7])};
    pf[u] = __builtin_bit_cast(bf16x8, w);
  }
}

// out[dt] += TileT[32 dt + lane%32, pos] * pf[pos, lane] over the 32 positions 32 T ..; off = rm_trans_off(lane).
template <int D, int T>
DEV void rm_mma_cols(uint32_t tile_addr, uint32_t off, const bf16x8 (&pf)[2], f32x16 (&out)[Dims<D>::DT]) {
  using X = Dims<D>;
  u32x2 vf[2][2][2];
  auto read_v = [&](auto dd) {
    constexpr int DTI = decltype(dd)::value;
    static_for<0, 2>([&](auto uu) {
      constexpr int U = decltype(uu)::value, OFF = T * 8192 + U * 4096;
      vf[DTI & 1][U][0] = ds_read_tr_at<OFF>(tile_addr + (off ^ ((4 * DTI) << 4)));
      vf[DTI & 1][U][1] = ds_read_tr_at<OFF + 2048>(tile_addr + (off ^ (((4 * DTI) ^ 2) << 4)));
    });
  };
  read_v(std::integral_constant<int, 0>{});
  static_for<0, X::DT>([&](auto dd) {
    constexpr int DTI = decltype(dd)::value;
    if constexpr (DTI + 1 < X::DT) read_v(std::integral_constant<int, DTI + 1>{});
    lds_wait<(DTI + 1 < X::DT) ? 4 : 0>();
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      tie(vf[DTI & 1][u][0]);
      tie(vf[DTI & 1][u][1]);
      const u32x4 a = {vf[DTI & 1][u][0][0], vf[DTI & 1][u][0][1], vf[DTI & 1][u][1][0], vf[DTI & 1][u][1][1]};
      out[DTI] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), pf[u], out[DTI], 0, 0, 0);
    }
  });
}

constexpr int RM_TILE = 16384;
using half0 = std::integral_constant<int, 0>;      // the halves of a tile of 64 positions
using half1 = std::integral_constant<int, 1>;

// Start of a score product over 32 tile positions: -inf where the causal mask hides the position from the lane's query or
// key (last: the largest tile row that stays, first: the smallest), so that the product itself carries the mask and no
// branch stands between its MFMAs and the first use of their sums.  The hardware does not hold back a use that comes too
// soon; the compiler keeps the distance by counting wait states, but it counts a block that two paths share along one of
// them only, and behind a few branches the shorter path can come out short (ROCm 7.2: 11 states of 12 behind an if with an
// if in both arms).  Branches as such are not unsafe: those behind products in this file (the mask and the maximum in
// attn_fwd_kernel, the rotation before the stores of both backward bodies) keep their distance on every path, as
// tests/test_mfma_distance.py finds on the assembly of all kernels, for the registers of LDS reads in flight as well.
DEV void start_scores(f32x16& acc, bool masked, int first, int last, int fh) {
#pragma unroll
  for (int v = 0; v < 16; ++v) acc[v] = 0.0f;
  if (masked) {
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = acc_row(v, fh) > last || acc_row(v, fh) < first ? -INFINITY : 0.0f;
  }
}
// ---- heads of 128, one wave per SIMD.  A tile of 64 positions is a chain of steps of two MFMAs: the row products of both
// halves (32 positions each), then the column products.  With one wave nothing else covers a wait, so the wave does it: the vector
// work of one half stands between the MFMAs of the other's, and fragments are read 3 or 4 steps before they are used.
// (4 x 4096 positions, 5 heads: 394 us with fragments read one batch ahead and the softmax between the products, 330 so; 2 x
// 4096, 4 heads 162 -> 146; 2 x 2048, 5 heads 76 -> 65.  A tile takes 4400 clocks, 2048 of them MFMAs.)
// The MFMAs are inline assembly, which says where their operands live: the running sums and the wave's own rows (its keys
// and values, or queries and gradients) in accumulation registers, scores in vector registers, where the softmax takes
// them from.  Left to the compiler all results go to accumulation registers and every score is copied.  It does not see
// these instructions' latency: results are used behind the reads and the MFMAs of the next step (checked on the
// assembly), running sums behind idle clocks of their own, and an operand that the vector ALU has just written gets two.
// The matrix pipe holds one MFMA beside the one at work: a pair of them, then other work, takes 82 clocks for the pair and 8
// multiply-adds, one MFMA and 4 of them twice takes 67.  So a step's other work is dealt out behind each of its MFMAs.
template <bool FIRST>
DEV void score_mfma(bf16x8 a, bf16x8 own, f32x16& sums) {        // FIRST: the sums' start has just been written
  if constexpr (FIRST) asm volatile("s_nop 1\n\tv_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(sums) : "v"(a), "a"(own));
  else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(sums) : "v"(a), "a"(own));
}
DEV void score_mfma_zero(bf16x8 a, bf16x8 own, f32x16& sums) { asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(sums) : "v"(a), "a"(own)); }
template <bool FIRST>
DEV void sums_mfma(bf16x8 a, bf16x8 p, f32x16& sums) {           // FIRST: the operand p has just been written
  if constexpr (FIRST) asm volatile("s_nop 1\n\tv_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(sums) : "v"(a), "v"(p));
  else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(sums) : "v"(a), "v"(p));
}
template <int N>
DEV void wait_for(u32x4& a, u32x4& b) { asm volatile("s_waitcnt lgkmcnt(%2)" : "+v"(a), "+v"(b) : "n"(N) : "memory"); }
template <int N>
DEV void wait_for(u32x2& a, u32x2& b, u32x2& c, u32x2& d) { asm volatile("s_waitcnt lgkmcnt(%4)" : "+v"(a), "+v"(b), "+v"(c), "+v"(d) : "n"(N) : "memory"); }

// The steps of a tile: 0 .. 7 and 8 .. 15 the row products of half 0 and 1 (one contraction step over d each), then four steps
// (d tiles) a column product.  A step's fragments are 2 reads (rows) or 4 (columns), issued behind the MFMAs of an earlier one;
// the dK/dV pass also reads the lse and D of 16 queries a lane, two reads for 4 queries, in front of them.
template <bool DKV>
struct BwdSteps {
  static constexpr int ROWS = 16, N = DKV ? 32 : 24;
  static constexpr int issued_at(int g) { return g < ROWS ? g - 4 : g - 3; }            // the step behind which g's reads stand; < 0: before the first
  static constexpr int group_of(int t) { for (int g = 0; g < N; ++g) if (issued_at(g) == t) return g; return -1; }
  static constexpr int stats_at(int t) { return !DKV ? -1 : t >= 0 && t < 4 ? t : t >= 11 && t <= 17 && t % 2 == 1 ? 4 + (t - 11) / 2 : -1; }
  static constexpr int reads(int g) { return g < ROWS ? 2 : 4; }
  static constexpr int stats_through(int t) { int n = 0; for (int u = 0; u <= t; ++u) n += stats_at(u) >= 0 ? 2 : 0; return n; }
  static constexpr int through_step(int t) { int n = stats_through(t); for (int g = 0; g < N; ++g) n += issued_at(g) <= t ? reads(g) : 0; return n; }
  static constexpr int through_group(int g) { int n = stats_through(issued_at(g)); for (int h = 0; h <= g; ++h) n += reads(h); return n; }
  static constexpr int behind(int g) { return through_step(g - 1) - through_group(g); } // reads that may still be in flight at step g
};

// an operand that stays in accumulation registers from here on
DEV void keep_in_acc(bf16x8 (&f)[8]) {
#pragma unroll
  for (int i = 0; i < 8; ++i) asm volatile("" : "+a"(f[i]));
}
// behind the loop: the last sums are as many clocks away from their MFMA as a use needs, and no copy of them is made before
template <int N>
DEV void settle(f32x16 (&acc)[N]) {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_nop 7\n\ts_nop 7");
  pin_acc(acc);
  __builtin_amdgcn_sched_barrier(0);
}

// The vector work of a half in steps of PER pairs of scores: the powers of the pairs to come, then what needs the powers taken a
// step before, so that neither waits for the other.
template <int K, int PER, class Half, class Powers>
DEV void powers_step(Half half, Powers&& powers) {
  constexpr int a0 = K == 0 ? 0 : (K + 1) * PER, a1 = (K + 2) * PER < 8 ? (K + 2) * PER : 8;
  static_for<(a0 < 8 ? a0 : 8), a1>([&](auto wc) { powers(half, wc); });
}
template <int K, int PER, class Half, class Grads>
DEV void grads_step(Half half, Grads&& grads) {
  constexpr int b0 = K == 0 ? 0 : (K - 1) * PER, b1 = K == 0 ? 0 : (K + 1) * PER == 8 ? 8 : K * PER;
  static_for<b0, b1>([&](auto wc) { grads(half, wc); });
}

// One tile.  rows_a, rows_b: LDS addresses of the tiles of the row products (with the own rows fa, fb; their sums are the two
// score accumulators sa, sb of each half); cols(c) gives the address, the operand and the sums of column product c (four steps).
// start() gives sa their start; powers(T, W) and grads(T, W) turn pair W of half T's scores into operands; stats(i) reads what
// they need for 4 queries; load(i) asks for piece i of the next tile, which costs 48 clocks where nothing stands beside it.
template <bool DKV, class Start, class Load, class Stats, class Powers, class Grads, class Cols>
DEV void bwd_tile(uint32_t rows_a, uint32_t rows_b, uint32_t off_rows, uint32_t off_cols, const bf16x8 (&fa)[8], const bf16x8 (&fb)[8],
                  f32x16 (&sa)[2], f32x16 (&sb)[2], Start&& start, Load&& load, Stats&& stats, Powers&& powers, Grads&& grads, Cols&& cols) {
  using S = BwdSteps<DKV>;
  u32x4 fr[5][2];
  u32x2 vf[4][2][2];
  auto read_group = [&](auto gc) {
    constexpr int G = decltype(gc)::value;
    if constexpr (G < S::ROWS) {
      constexpr int T = G / 8, KS = G % 8;
      fr[G % 5][0] = ds_read_b128_at<T * 8192>(rows_a + (off_rows ^ (KS << 5)));
      fr[G % 5][1] = ds_read_b128_at<T * 8192>(rows_b + (off_rows ^ (KS << 5)));
    } else {
      constexpr int C = (G - S::ROWS) / 4, DTI = (G - S::ROWS) % 4, T = DKV ? C / 2 : C;
      const uint32_t tile = cols(std::integral_constant<int, C>{}, nullptr);
      static_for<0, 2>([&](auto uu) {
        constexpr int U = decltype(uu)::value, OFF = T * 8192 + U * 4096;
        vf[G % 4][U][0] = ds_read_tr_at<OFF>(tile + (off_cols ^ ((4 * DTI) << 4)));
        vf[G % 4][U][1] = ds_read_tr_at<OFF + 2048>(tile + (off_cols ^ (((4 * DTI) ^ 2) << 4)));
      });
    }
  };
  static_for<0, 4>([&](auto g) { read_group(g); });
  start();
  static_for<0, S::N>([&](auto gc) {
    constexpr int G = decltype(gc)::value;
    static_assert(S::behind(G) <= 15, "the LDS counter has four bits");
    __builtin_amdgcn_sched_barrier(0);
    constexpr int STEP = G >= 16 ? G - 16 : G - 8, PER = G >= 16 && !DKV ? 2 : 1;      // the softmax's step of a half
    constexpr bool SOFTMAX = G >= 8 && G < (DKV ? 24 : 20);
    using half = std::integral_constant<int, G >= 16 ? 1 : 0>;
    auto beside = [&] {
      __builtin_amdgcn_sched_barrier(0);
      if constexpr (S::stats_at(G) >= 0) stats(std::integral_constant<int, S::stats_at(G)>{});
      if constexpr (S::group_of(G) >= 0) read_group(std::integral_constant<int, S::group_of(G)>{});
      if constexpr (G < 8) load(gc);
      if constexpr (G == 8 || G == 16) {          // a half's scores: the distance to their first use
        asm volatile("s_nop 7");
        __builtin_amdgcn_sched_barrier(0);
      }
      if constexpr (SOFTMAX) powers_step<STEP, PER>(half{}, powers);
      __builtin_amdgcn_sched_barrier(0);
    };
    if constexpr (G < S::ROWS) {
      constexpr int T = G / 8, KS = G % 8;
      wait_for<S::behind(G)>(fr[G % 5][0], fr[G % 5][1]);
      score_mfma<KS == 0>(__builtin_bit_cast(bf16x8, fr[G % 5][0]), fa[KS], sa[T]);
      beside();
      if constexpr (KS == 0) score_mfma_zero(__builtin_bit_cast(bf16x8, fr[G % 5][1]), fb[KS], sb[T]);
      else score_mfma<false>(__builtin_bit_cast(bf16x8, fr[G % 5][1]), fb[KS], sb[T]);
    } else {
      constexpr int C = (G - S::ROWS) / 4, DTI = (G - S::ROWS) % 4;
      u32x2 (&v)[2][2] = vf[G % 4];
      wait_for<S::behind(G)>(v[0][0], v[0][1], v[1][0], v[1][1]);
      cols(std::integral_constant<int, C>{}, [&](const uint32_t (&w)[8], auto& sums) {
        const u32x4 a0 = {v[0][0][0], v[0][0][1], v[0][1][0], v[0][1][1]}, a1 = {v[1][0][0], v[1][0][1], v[1][1][0], v[1][1][1]};
        sums_mfma<DTI == 0>(__builtin_bit_cast(bf16x8, a0), __builtin_bit_cast(bf16x8, u32x4{w[0], w[1], w[2], w[3]}), sums[DTI]);
        beside();
        sums_mfma<DTI == 0>(__builtin_bit_cast(bf16x8, a1), __builtin_bit_cast(bf16x8, u32x4{w[4], w[5], w[6], w[7]}), sums[DTI]);
      });
    }
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (SOFTMAX) grads_step<STEP, PER>(half{}, grads);
    __builtin_amdgcn_sched_barrier(0);
  });
}

// the same for sums in vector registers
template <int N>
DEV void settle_v(f32x16 (&acc)[N]) {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_nop 7\n\ts_nop 7");
#pragma unroll
  for (int i = 0; i < N; ++i) asm volatile("" : "+v"(acc[i]));
  __builtin_amdgcn_sched_barrier(0);
}

// ------------------------------------------------------------------------------------- forward
// One workgroup = 128 queries of one (batch element, head): 4 waves x 32 queries.  A tile of 64 keys is a chain of scores, softmax and
// output, and the longest workgroup's tiles are the launch's time where the chip is not full many times over.  So a wave
// works on two tiles at once: while the scores of tile j + 1 are formed the softmax of tile j ends, and while the output products
// of tile j run that of tile j + 1 begins.  A step is two MFMAs with vector work dealt out behind each.
// What bounds a wave alone is that it issues one instruction of any kind every 4 to 8 clocks (2^x 8, a dependent addition 8): some
// 400 a tile, so LDS places are constants of the instructions (the loop is written for two tiles) and the products, the
// waits and the powers are most of what is left.  With two workgroups on a compute unit it is the LDS: each wave reads all of K and V.
// K and V tiles travel HBM/L2 -> LDS with buffer_load ... lds into two places each: K as contraction-contiguous [kv][32 d]
// sub-tiles, V as row-major [32 kv][128 d] ones read back with the transposing LDS read in accumulator-row order, so P feeds P V
// straight from registers.  MFMAs are inline assembly on vector registers only: with accumulation registers in use the compiler
// halves the 256 that two waves per SIMD leave each.
// (us, with each tile's three parts one after the other and so: heads of 128, 2 x 4096 positions, 4 heads 82 -> 63, 4 x 2048, 5 heads
// 46 -> 39, 4 x 4096, 5 heads 104 -> 100, 44 x 448, 7 heads 52 -> 51; heads of 80, 8 x 2048, 4 heads 43 -> 37, 6 x 1003, 4 heads
// 20.9 -> 17.6; heads of 64, 2 x 2048, 5 heads 32 -> 27.  44 x 448, 7 heads of 64 would take 27.5 for 26 and keep the serial form below.
// One wave per SIMD with deeper rings and Q and K in accumulation registers: 71, 41 and 122 for the first three.)
template <int D>
struct FwdSteps {
  static constexpr int KS = Dims<D>::KSTEPS, NV = 2 * Dims<D>::DT;                   // steps of the scores and of the output, two MFMAs each
  static constexpr int EARLY = D == 128 ? 10 : 8;                                    // pairs of probabilities (of 16) taken beside the output products
  static constexpr int AK = D == 128 ? 2 : 3, AV = AK;                                               // steps ahead that fragments are read
  // reads in flight that step `at` (scores 0 .. KS - 1, then output) may leave so: those of the steps behind it
  static constexpr int reads(int at) { return at < KS ? 2 : at < KS + NV ? 4 : 0; }
  static constexpr int issued(int at) { return at < KS ? at - AK : at - AV; }          // the step beside which `at`'s reads stand
  static constexpr int behind(int at) {
    int n = 0;
    for (int k = at + 1; k < KS + NV; ++k) n += issued(k) < at ? reads(k) : 0;
    return n;
  }
};
// All in vector registers; ZERO: the first product of a sum.  The wait for the fragments stands in the same statement.
template <bool ZERO, int WAIT>
DEV void fwd_score_mfma(const u32x4& k, bf16x8 q, f32x16& t) {
  if constexpr (WAIT >= 0) {
    if constexpr (ZERO) asm volatile("s_waitcnt lgkmcnt(%3)\n\tv_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(t) : "v"(k), "v"(q), "n"(WAIT));
    else asm volatile("s_waitcnt lgkmcnt(%3)\n\tv_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(t) : "v"(k), "v"(q), "n"(WAIT));
  } else {
    if constexpr (ZERO) asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, 0" : "=&v"(t) : "v"(k), "v"(q));
    else asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(t) : "v"(k), "v"(q));
  }
}
DEV void fwd_output_mfma(const u32x4& v, const u32x4& p, f32x16& o) { asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+v"(o) : "v"(v), "v"(p)); }
// a value is formed here, and not behind the branches that follow, or ahead of the loop
template <class T>
DEV void here(T& v) { asm volatile("" : "+v"(v)); }
DEV void idle8() {
  asm volatile("s_nop 7");
  __builtin_amdgcn_sched_barrier(0);
}
// both transposing reads of 16 keys into the halves of one fragment
template <int OFF>
DEV void read_v_frag(uint32_t addr, u32x2& a, u32x2& b) {
  a = ds_read_tr_at<OFF>(addr);
  b = ds_read_tr_at<OFF + 2048>(addr);
}

template <int D>
DEV void attn_fwd_body(const AttnArgs& p, uint8_t* smem) {
  using X = Dims<D>;
  using S = FwdSteps<D>;
  constexpr int DS = (D + 31) / 32;                 // 32-wide d sub-tiles of K
  constexpr int K_BYTES = DS * 4096, V_BYTES = 2 * 8192;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int fr = lane & 31, fh = lane >> 5;
  const int s = p.seq;
  const int nqb = (s + 127) / 128;
  int pos, group;
  if (!ranked_item(nqb, p.heads * p.batch, pos, group)) return;
  const int qb = nqb - 1 - pos;                     // longest rows first
  const int hh = group % p.heads, bi = group / p.heads;
  const int qw0 = qb * 128 + wave * 32, qpos = qw0 + fr;
  const long ld = p.ld;
  const bf16_t* tok0 = static_cast<const bf16_t*>(p.qkv) + (long)bi * s * ld;
  const int hl = p.heads * D;
  const int ntiles = (min(qb * 128 + 128, s) + 63) / 64;
  const int mine = min((qw0 + 31) / 64 + 1, ntiles);          // tiles that this wave's queries see; the others see at most one more

  // loads: a wave's pieces of a tile.  The tile is advanced in the buffer resource, whose extent ends with the last tile or
  // row that is needed: what lies beyond gives zeros.
  DmaLoader<64, 4, false> ldK;
  DmaLoader<128, 4, true> ldV;
  ldK.init_kc((int)ld, 0, 1 << 30, wave, lane);
  ldV.init_ks((int)ld, IdentityCols{0, D}, wave, lane);
  uint32_t at_k[DS], at_v[4];
#pragma unroll
  for (int c = 0; c < DS; ++c) at_k[c] = c * 32 + ldK.kofs < D ? ldK.base[0] + c * 64 : BUF_OOB;
#pragma unroll
  for (int i = 0; i < 4; ++i) at_v[i] = ldV.base[i & 1] + (uint32_t)((i >> 1) * 32) * (uint32_t)ld * 2u;
  const int step = attention_tile_bytes(ld);
  const char* next_k = reinterpret_cast<const char*>(tok0 + hl + hh * D);
  const char* next_v = reinterpret_cast<const char*>(tok0 + 2 * hl + hh * D);
  int left_k = attention_view_bytes(min(ntiles * 64, s), (int)ld, D), left_v = left_k;
  auto load_k = [&](int c, buf_rsrc rs, int slot) { __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, LDS_PTR(smem + slot * K_BYTES + c * 4096 + wave * 1024), 16, at_k[c], 0, 0, 0); };
  auto load_v = [&](int i, buf_rsrc rs, int slot) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, LDS_PTR(smem + 2 * K_BYTES + slot * V_BYTES + (i >> 1) * 8192 + (wave * 2 + (i & 1)) * 1024), 16, at_v[i], 0, 0, 0);
  };
  auto advance_k = [&] { next_k += step; left_k = attention_left_behind(left_k, step); };
  auto advance_v = [&] { next_v += step; left_v = attention_left_behind(left_v, step); };
  auto fill_k = [&](int slot) {
    const buf_rsrc rs = make_rsrc(next_k, left_k);
#pragma unroll
    for (int c = 0; c < DS; ++c) load_k(c, rs, slot);
    advance_k();
  };
  auto fill_v = [&](int slot) {
    const buf_rsrc rs = make_rsrc(next_v, left_v);
#pragma unroll
    for (int i = 0; i < 4; ++i) load_v(i, rs, slot);
    advance_v();
  };
  bf16x8 qf[X::KSTEPS];
  load_row_frags<D>(tok0 + hh * D, ld, qpos, s, fh, qf);
  fill_k(0); fill_v(0); fill_k(1);

  // per-lane LDS addresses: K fragment (row lane%32, chunk 2*step + lane/32) and V^T fragment rows d
  const uint32_t lds = lds_addr(smem);
  const uint32_t offK[2] = {lds + kc_frag_off(lane, 0), lds + kc_frag_off(lane, 1)};
  uint32_t offV[X::DT];
  {
    const int sl = lane & 15, nh = (lane >> 4) & 1;
    const int kr = 4 * fh + (sl >> 2);
#pragma unroll
    for (int dt = 0; dt < X::DT; ++dt) offV[dt] = lds + (uint32_t)(kr * 256 + ((dt ^ (kr & 3)) << 6) + (16 * nh + 4 * (sl & 3)) * 2);
  }
  f32x16 o[X::DT], sT[2][2];                        // sT[j & 1]: scores of tile j, then their powers
#pragma unroll
  for (int dt = 0; dt < X::DT; ++dt)
#pragma unroll
    for (int v = 0; v < 16; ++v) o[dt][v] = 0.0f;
  uint32_t pw[16];                                  // P, packed: pair w of the 32 scores
  float m = -INFINITY, l = 0.0f, alpha = 1.0f, rs = 0.0f, mx = 0.0f;
  uint64_t moved = 0;                               // queries whose maximum moved with the tile
  const float sc = p.scale * LOG2E;

  u32x4 kf[S::AK + 1][2];
  u32x2 vf[S::AV + 1][2][2];
  auto read_k = [&](auto gc, auto slot) {
    constexpr int G = decltype(gc)::value, OFF = decltype(slot)::value * K_BYTES + (G >> 1) * 4096;
    kf[G % (S::AK + 1)][0] = ds_read_b128_at<OFF>(offK[G & 1]);
    kf[G % (S::AK + 1)][1] = ds_read_b128_at<OFF + 2048>(offK[G & 1]);
  };
  auto read_v = [&](auto hc, auto slot) {           // step h: d tile h / 2, 32 keys of half h % 2
    constexpr int H = decltype(hc)::value, OFF = 2 * K_BYTES + decltype(slot)::value * V_BYTES + (H & 1) * 8192;
    read_v_frag<OFF>(offV[H / 2], vf[H % (S::AV + 1)][0][0], vf[H % (S::AV + 1)][0][1]);
    read_v_frag<OFF + 4096>(offV[H / 2], vf[H % (S::AV + 1)][1][0], vf[H % (S::AV + 1)][1][1]);
  };
  // reads that stand beside step `at`: K from place sk, V from place sv
  auto reads_beside = [&](auto at, auto sk, auto sv) {
    static_for<0, S::KS>([&](auto g) { if constexpr (S::issued(decltype(g)::value) == decltype(at)::value) read_k(g, sk); });
    static_for<0, S::NV>([&](auto h) { if constexpr (S::issued(S::KS + decltype(h)::value) == decltype(at)::value) read_v(h, sv); });
  };
  auto score_step = [&](auto gc, auto&& beside, f32x16 (&t)[2], auto waits) {
    constexpr int G = decltype(gc)::value;
    u32x4 (&k)[2] = kf[G % (S::AK + 1)];
    static_for<0, 2>([&](auto tc) {
      constexpr int T = decltype(tc)::value;
      fwd_score_mfma<G == 0, T == 0 ? decltype(waits)::value : -1>(k[T], qf[G], t[T]);
      __builtin_amdgcn_sched_barrier(0);
      beside(tc);
      __builtin_amdgcn_sched_barrier(0);
    });
  };
  auto output_step = [&](auto hc, auto&& beside, auto waits) {
    constexpr int H = decltype(hc)::value;
    u32x2 (&v)[2][2] = vf[H % (S::AV + 1)];
    static_for<0, 2>([&](auto uc) {
      constexpr int U = decltype(uc)::value, W = 8 * (H & 1) + 4 * U;
      if constexpr (U == 0) wait_for<decltype(waits)::value>(v[0][0], v[0][1], v[1][0], v[1][1]);
      const u32x4 a = {v[U][0][0], v[U][0][1], v[U][1][0], v[U][1][1]}, b = {pw[W], pw[W + 1], pw[W + 2], pw[W + 3]};
      fwd_output_mfma(a, b, o[H / 2]);
      __builtin_amdgcn_sched_barrier(0);
      beside(uc);
      __builtin_amdgcn_sched_barrier(0);
    });
  };
  // ---- online softmax; a lane owns one query (both lane halves: the two key halves of each 8)
  auto maximum = [&](f32x16 (&t)[2], int j) {
    if (j == mine - 1) {                            // the tile meets the diagonal: mask keys after the query
      int last = qpos - j * 64;                     // (opaque: 32 comparisons of the last tile, kept from the start, would take 64 scalar registers)
      here(last);
#pragma unroll
      for (int T = 0; T < 2; ++T)
#pragma unroll
        for (int v = 0; v < 16; ++v)
          if (32 * T + acc_row(v, fh) > last) t[T][v] = -INFINITY;
    }
    mx = -INFINITY;
#pragma unroll
    for (int T = 0; T < 2; ++T)
#pragma unroll
      for (int v = 0; v < 16; ++v) mx = fmaxf(mx, t[T][v]);
  };
  auto statistics = [&] {
    mx = fmaxf(mx, other_half(mx)) * sc;            // scores scaled to the log2 domain (sc > 0)
    const float m_new = fmaxf(m, mx);               // finite: key 0 is visible to every query
    moved = __builtin_amdgcn_ballot_w64(m_new != m);           // rescale only when some query's maximum moved
    if (moved) {
      alpha = exp2_raw(m - m_new);
      l *= alpha;
      m = m_new;
    }
    rs = 0.0f;
  };
  auto rescale = [&] {
    if (moved) {
#pragma unroll
      for (int dt = 0; dt < X::DT; ++dt)
#pragma unroll
        for (int v = 0; v < 16; ++v) o[dt][v] *= alpha;
    }
  };
  auto power = [&](f32x16 (&t)[2], auto wc) {       // pair w of the powers, in the place of their scores
    constexpr int T = decltype(wc)::value / 8, V = decltype(wc)::value % 8 * 2;
    float e0 = exp2_raw(t[T][V] * sc - m), e1 = exp2_raw(t[T][V + 1] * sc - m);
    rs += e0;
    rs += e1;
    here(e0);
    here(e1);
    here(rs);
    t[T][V] = e0;
    t[T][V + 1] = e1;
  };
  auto pack = [&](f32x16 (&t)[2], auto wc) {
    constexpr int W = decltype(wc)::value, T = W / 8, V = W % 8 * 2;
    pw[W] = pack_bf16(t[T][V], t[T][V + 1]);
    here(pw[W]);
  };
  // vector work of score step G of the tile after t's: the end of t's softmax
  constexpr int LATE = 16 - S::EARLY;
  auto beside_scores = [&](auto gc, auto half, f32x16 (&t)[2]) {
    constexpr int G = decltype(gc)::value, H = 2 * G + decltype(half)::value, NH = 2 * S::KS;
    if constexpr (H == 5) rescale();
    static_for<S::EARLY * H / NH, S::EARLY * (H + 1) / NH>([&](auto w) { pack(t, w); });
    static_for<S::EARLY + LATE * H / NH, S::EARLY + LATE * (H + 1) / NH>([&](auto w) { power(t, w); pack(t, w); });
    if constexpr (H == NH - 1) { l += rs; here(l); }
  };
  // vector work of output step h: the beginning of the softmax of tile j
  auto beside_output = [&](auto hc, auto half, f32x16 (&t)[2], int j) {
    constexpr int H = decltype(hc)::value, Q = 2 * (H - 2) + decltype(half)::value, NQ = 2 * (S::NV - 2);
    if constexpr (H == 1 && decltype(half)::value == 0) { idle8(); maximum(t, j); }
    if constexpr (H == 1 && decltype(half)::value == 1) statistics();
    if constexpr (H >= 2) static_for<S::EARLY * Q / NQ, S::EARLY * (Q + 1) / NQ>([&](auto w) { power(t, w); });
  };

  // scores of tile 0, and the beginning of its softmax
  wait_vmcnt<4 + DS>();
  __builtin_amdgcn_s_barrier();
  static_for<0, S::AK>([&](auto g) { read_k(g, half0{}); });
  static_for<0, S::KS>([&](auto gc) {
    constexpr int G = decltype(gc)::value, NEXT = G + S::AK, LEFT = S::KS - 1 - G;
    score_step(gc, [&](auto half) {
      if constexpr (decltype(half)::value == 0 && NEXT < S::KS) read_k(std::integral_constant<int, (NEXT < S::KS ? NEXT : 0)>{}, half0{});
    }, sT[0], std::integral_constant<int, 2 * (LEFT < S::AK - 1 ? LEFT : S::AK - 1)>{});
  });
  wait_vmcnt<0>();
  __builtin_amdgcn_s_barrier();
  idle8();
  maximum(sT[0], 0);
  statistics();
  moved = 0;                                        // there is no output yet to rescale
  static_for<0, S::EARLY>([&](auto w) { power(sT[0], w); });

  auto both = [&](auto cur, int j) {                // scores of tile j + 1, output of tile j
    constexpr int C = decltype(cur)::value;
    using other = std::integral_constant<int, C ^ 1>;
    f32x16 (&now)[2] = sT[C];
    f32x16 (&nxt)[2] = sT[C ^ 1];
    const buf_rsrc rk = make_rsrc(next_k, left_k), rv = make_rsrc(next_v, left_v);
    static_for<-S::AK, 0>([&](auto at) { reads_beside(at, other{}, cur); });
    static_for<0, S::KS>([&](auto gc) {
      constexpr int G = decltype(gc)::value;
      score_step(gc, [&](auto half) {
        constexpr int Q = 2 * G + decltype(half)::value, N = 2 * S::KS, L = DS + 4;
        if constexpr (decltype(half)::value == 0) { reads_beside(gc, other{}, cur); __builtin_amdgcn_sched_barrier(0); }
        static_for<L * Q / N, L * (Q + 1) / N>([&](auto ic) {      // K of tile j + 2 in the place of tile j's, V of tile j + 1
          constexpr int I = decltype(ic)::value;
          if constexpr (I < DS) load_k(I, rk, C); else load_v(I - DS, rv, C ^ 1);
        });
        beside_scores(gc, half, now);
      }, nxt, std::integral_constant<int, S::behind(G)>{});
    });
    advance_k();
    advance_v();
    static_for<0, S::NV>([&](auto hc) {
      constexpr int H = decltype(hc)::value;
      output_step(hc, [&](auto half) {
        if constexpr (decltype(half)::value == 0) { reads_beside(std::integral_constant<int, S::KS + H>{}, other{}, cur); __builtin_amdgcn_sched_barrier(0); }
        beside_output(hc, half, nxt, j + 1);
      }, std::integral_constant<int, S::behind(S::KS + H)>{});
    });
    wait_vmcnt<0>();
    __builtin_amdgcn_s_barrier();
  };
  int j = 0;
  for (; j + 2 < mine; j += 2) {
    both(half0{}, j);
    both(half1{}, j + 1);
  }
  auto end = [&](auto cur) {                        // the last tile: the end of its softmax, its output
    constexpr int C = decltype(cur)::value;
    if (mine < ntiles) fill_v(C ^ 1);               // the tile that the other waves' queries still see
    static_for<0, S::AV>([&](auto h) { read_v(h, cur); });
    settle_v(o);
    static_for<0, S::KS>([&](auto gc) { beside_scores(gc, half0{}, sT[C]); beside_scores(gc, half1{}, sT[C]); });
    idle8();
    static_for<0, S::NV>([&](auto hc) {
      constexpr int H = decltype(hc)::value;
      output_step(hc, [&](auto half) {
        if constexpr (decltype(half)::value == 0 && H + S::AV < S::NV) read_v(std::integral_constant<int, H + S::AV < S::NV ? H + S::AV : 0>{}, cur);
      }, std::integral_constant<int, (S::NV - 1 - H < S::AV - 1 ? S::NV - 1 - H : S::AV - 1) * 4>{});
    });
    settle_v(o);
  };
  if (j + 1 < mine) {
    both(half0{}, j);
    end(half1{});
  } else {
    end(half0{});
  }
  wait_vmcnt<0>();                                  // what was asked for ahead lands before the LDS is another workgroup's
  if (mine < ntiles) __builtin_amdgcn_s_barrier();
  l += other_half(l);
  if (qpos < s) {
    bf16_t* out = static_cast<bf16_t*>(p.ctx) + ((long)bi * s + qpos) * p.ld_ctx + hh * D;
    store_transposed<D>(o, 1.0f / l, out, fh);
    if (fh == 0) p.lse[((long)bi * p.heads + hh) * s + qpos] = (m + log2f(l)) * LN2;
  }
}
template <int D>
__global__ __launch_bounds__(256, 2)
void attn_fwd_kernel(const AttnArgs p) {
  extern __shared__ __align__(1024) uint8_t smem[];
  attn_fwd_body<D>(p, smem);
}

// The same sums with the three parts of a tile one after the other: 120 registers and 48 KB of LDS for heads of 64, so that three
// workgroups share a compute unit, and nothing in front of the first tile's scores that a lone tile does not need.  What bounds a
// wave is that chain; attention_fwd_serial (attention.h) says where it is the faster one all the same, with both sides measured.  K and
// V in two places of 64 keys each, loaded together a tile ahead.
template <int D>
__global__ __launch_bounds__(256, 2)
void attn_fwd_serial_kernel(const AttnArgs p) {
  using X = Dims<D>;
  constexpr int DS = (D + 31) / 32;                 // 32-wide d sub-tiles of K
  constexpr int K_BYTES = DS * 4096;                // [DS][64 kv][32 d]
  constexpr int V_BYTES = 2 * 8192;                 // [2][32 kv][128 d]
  constexpr int STAGE = K_BYTES + V_BYTES;
  constexpr int NB = (X::KSTEPS + 3) / 4;           // batches of up to 4 contraction steps over d
  extern __shared__ __align__(1024) uint8_t smem[];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int fr = lane & 31, fh = lane >> 5;
  const int s = p.seq;
  const int nqb = (s + 127) / 128;
  int pos, group;
  if (!ranked_item(nqb, p.heads * p.batch, pos, group)) return;
  const int qb = nqb - 1 - pos;                     // longest rows first
  const int hh = group % p.heads, bi = group / p.heads;
  const int qw0 = qb * 128 + wave * 32, qpos = qw0 + fr;
  const long ld = p.ld;
  const bf16_t* tok0 = static_cast<const bf16_t*>(p.qkv) + (long)bi * s * ld;
  const int hl = p.heads * D;
  const long view_bytes = ((long)(s - 1) * ld + D) * 2;
  const buf_rsrc rsK = make_rsrc(tok0 + hl + hh * D, view_bytes);
  const buf_rsrc rsV = make_rsrc(tok0 + 2 * hl + hh * D, view_bytes);

  bf16x8 qf[X::KSTEPS];
  load_row_frags<D>(tok0 + hh * D, ld, qpos, s, fh, qf);

  DmaLoader<64, 4, false> ldK;
  DmaLoader<128, 4, true> ldV;
  ldK.init_kc((int)ld, 0, 1 << 30, wave, lane);       // rows past the sequence end fall outside the extent
  ldV.init_ks((int)ld, IdentityCols{0, D}, wave, lane);
  auto issue_tile = [&](int j) {
    uint8_t* st = smem + (j & 1) * STAGE;
    const int kv0 = j * 64;
#pragma unroll
    for (int c = 0; c < DS; ++c) ldK.issue(rsK, st + c * 4096, c * 32, D, wave, (uint32_t)kv0 * (uint32_t)ld * 2u);
#pragma unroll
    for (int h2 = 0; h2 < 2; ++h2) ldV.issue(rsV, st + K_BYTES + h2 * 8192, kv0 + 32 * h2, 0, wave);
  };

  // per-lane LDS offsets: K fragment (row lane%32, chunk 2*step + lane/32) and V^T fragment rows d
  const uint32_t offK0 = kc_frag_off(lane, 0), offK1 = kc_frag_off(lane, 1);
  uint32_t offV[X::DT];
  {
    const int sl = lane & 15, nh = (lane >> 4) & 1;
    const int kr = 4 * fh + (sl >> 2);
#pragma unroll
    for (int dt = 0; dt < X::DT; ++dt)
      offV[dt] = (uint32_t)(kr * 256 + ((dt ^ (kr & 3)) << 6) + (16 * nh + 4 * (sl & 3)) * 2 + K_BYTES);
  }

  const int q_end = min(qb * 128 + 128, s);
  const int ntiles = (q_end + 63) / 64;
  f32x16 o[X::DT];
#pragma unroll
  for (int dt = 0; dt < X::DT; ++dt)
#pragma unroll
    for (int v = 0; v < 16; ++v) o[dt][v] = 0.0f;
  float m = -INFINITY, l = 0.0f;
  const float sc = p.scale * LOG2E;
  const uint32_t smem_base = lds_addr(smem);

  issue_tile(0);
  for (int j = 0; j < ntiles; ++j) {
    wait_vmcnt<0>();                                  // tile j has landed (this wave's part)
    __builtin_amdgcn_s_barrier();                     // ... everybody's part; the other stage is free
    if (j + 1 < ntiles) issue_tile(j + 1);
    const int kv0 = j * 64;
    if (kv0 > qw0 + 31) continue;                     // every key of the tile is masked for this wave
    const uint32_t st = smem_base + (j & 1) * STAGE;

    // ---- S^T[kv, q] = K Q^T: batches of 4 contraction steps, next batch's reads in flight
    f32x16 sT[2];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int v = 0; v < 16; ++v) sT[t][v] = 0.0f;
    u32x4 kf[2][4][2];
    auto read_batch = [&](auto bb) {
      constexpr int B = decltype(bb)::value;
      static_for<0, 4>([&](auto kk) {
        constexpr int KS = B * 4 + decltype(kk)::value;
        if constexpr (KS < X::KSTEPS) {
          const uint32_t a = st + ((KS & 1) ? offK1 : offK0);
          kf[B & 1][decltype(kk)::value][0] = ds_read_b128_at<(KS >> 1) * 4096>(a);
          kf[B & 1][decltype(kk)::value][1] = ds_read_b128_at<(KS >> 1) * 4096 + 2048>(a);
        }
      });
    };
    read_batch(std::integral_constant<int, 0>{});
    static_for<0, NB>([&](auto bb) {
      constexpr int B = decltype(bb)::value;
      constexpr int NEXT = (B + 1 < NB) ? ((X::KSTEPS - 4 * (B + 1)) < 4 ? (X::KSTEPS - 4 * (B + 1)) : 4) * 2 : 0;
      if constexpr (B + 1 < NB) read_batch(std::integral_constant<int, B + 1>{});
      lds_wait<NEXT>();
      static_for<0, 4>([&](auto kk) {
        constexpr int KS = B * 4 + decltype(kk)::value;
        if constexpr (KS < X::KSTEPS) {
          tie(kf[B & 1][decltype(kk)::value][0]);
          tie(kf[B & 1][decltype(kk)::value][1]);
#pragma unroll
          for (int t = 0; t < 2; ++t)
            sT[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kf[B & 1][decltype(kk)::value][t]),
                                                            qf[KS], sT[t], 0, 0, 0);
        }
      });
    });

    // ---- online softmax; a lane owns one query (both lane halves: the two key halves of each 8)
    float mx = -INFINITY;
    if (kv0 + 63 > qw0) {                             // tile touches the diagonal: mask keys after the query
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          if (kv0 + 32 * t + acc_row(v, fh) > qpos) sT[t][v] = -INFINITY;
          mx = fmaxf(mx, sT[t][v]);
        }
    } else {
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int v = 0; v < 16; ++v) mx = fmaxf(mx, sT[t][v]);
    }
    mx = fmaxf(mx, other_half(mx)) * sc;       // scores scaled to the log2 domain (sc > 0)
    const float m_new = fmaxf(m, mx);                  // finite: key 0 is visible to every query
    if (__builtin_amdgcn_ballot_w64(m_new != m) != 0) {   // rescale only when some query's maximum moved
      const float alpha = exp2_raw(m - m_new);
      l *= alpha;
#pragma unroll
      for (int dt = 0; dt < X::DT; ++dt)
#pragma unroll
        for (int v = 0; v < 16; ++v) o[dt][v] *= alpha;
      m = m_new;
    }
    float rs = 0.0f;
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const float e = exp2_raw(sT[t][v] * sc - m);
        sT[t][v] = e;
        rs += e;
      }
    l += rs;
    bf16x8 pf[4];
#pragma unroll
    for (int s4 = 0; s4 < 4; ++s4) {
      const int t = s4 >> 1, u = s4 & 1;
      u32x4 w = {pack_bf16(sT[t][8 * u + 0], sT[t][8 * u + 1]), pack_bf16(sT[t][8 * u + 2], sT[t][8 * u + 3]),
                 pack_bf16(sT[t][8 * u + 4], sT[t][8 * u + 5]), pack_bf16(sT[t][8 * u + 6], sT[t][8 * u + 7])};
      pf[s4] = __builtin_bit_cast(bf16x8, w);
    }

    // ---- O^T[d, q] += V^T P^T, one 32-row d tile at a time, next tile's reads in flight
    u32x2 vf[2][4][2];
    auto read_v = [&](auto dd) {
      constexpr int DTI = decltype(dd)::value;
      static_for<0, 4>([&](auto ss) {
        constexpr int S4 = decltype(ss)::value;
        constexpr int OFF = (S4 >> 1) * 8192 + (S4 & 1) * 4096;
        vf[DTI & 1][S4][0] = ds_read_tr_at<OFF>(st + offV[DTI]);
        vf[DTI & 1][S4][1] = ds_read_tr_at<OFF + 2048>(st + offV[DTI]);
      });
    };
    read_v(std::integral_constant<int, 0>{});
    static_for<0, X::DT>([&](auto dd) {
      constexpr int DTI = decltype(dd)::value;
      if constexpr (DTI + 1 < X::DT) read_v(std::integral_constant<int, DTI + 1>{});
      lds_wait<(DTI + 1 < X::DT) ? 8 : 0>();
#pragma unroll
      for (int s4 = 0; s4 < 4; ++s4) {
        tie(vf[DTI & 1][s4][0]);
        tie(vf[DTI & 1][s4][1]);
        const u32x4 a = {vf[DTI & 1][s4][0][0], vf[DTI & 1][s4][0][1], vf[DTI & 1][s4][1][0], vf[DTI & 1][s4][1][1]};
        o[DTI] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), pf[s4], o[DTI], 0, 0, 0);
      }
    });
  }
  l += other_half(l);
  if (qpos < s) {
    bf16_t* out = static_cast<bf16_t*>(p.ctx) + ((long)bi * s + qpos) * p.ld_ctx + hh * D;
    store_transposed<D>(o, 1.0f / l, out, fh);
    if (fh == 0) p.lse[((long)bi * p.heads + hh) * s + qpos] = (m + log2f(l)) * LN2;
  }
}

// ------------------------------------------------------------------------------------- dQ pass
template <int D>
DEV void attn_bwd_dq_body(const AttnArgs& p, uint8_t* smem, int qb, int hh, int bi) {
  using X = Dims<D>;
  constexpr int STAGE = 2 * RM_TILE;                      // K tile, V tile (64 keys each)
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int fr = lane & 31, fh = lane >> 5;
  const int s = p.seq;
  const int qw0 = qb * 128 + wave * 32, qpos = qw0 + fr;
  const long ld = p.ld;
  const bf16_t* tok0 = static_cast<const bf16_t*>(p.qkv) + (long)bi * s * ld;
  const int hl = p.heads * D;
  const long view_bytes = ((long)(s - 1) * ld + D) * 2;
  const buf_rsrc rsK = make_rsrc(tok0 + hl + hh * D, view_bytes);
  const buf_rsrc rsV = make_rsrc(tok0 + 2 * hl + hh * D, view_bytes);

  bf16x8 qf[X::KSTEPS], dof[X::KSTEPS];
  load_row_frags<D>(tok0 + hh * D, ld, qpos, s, fh, qf);
  load_row_frags<D>(static_cast<const bf16_t*>(p.dctx) + (long)bi * s * p.ld_ctx + hh * D, p.ld_ctx, qpos, s, fh, dof);
  if constexpr (D == 128) { keep_in_acc(qf); keep_in_acc(dof); }
  const long stat = ((long)bi * p.heads + hh) * s + qpos;
  const float lse2 = qpos < s ? p.lse[stat] * LOG2E : INFINITY;
  const float dq_dot = qpos < s ? p.dot[stat] : 0.0f;

  RmLoader ldr;
  ldr.init((int)ld, D, wave, lane);
  auto issue_tile = [&](int j) {
    uint8_t* st = smem + (j & 1) * STAGE;
    const uint32_t ro = (uint32_t)(j * 64) * (uint32_t)ld * 2u;
    ldr.issue(rsK, st, ro, wave);
    ldr.issue(rsV, st + RM_TILE, ro, wave);
  };
  const uint32_t offP = rm_plain_off(lane), offT = rm_trans_off(lane);

  const int q_end = min(qb * 128 + 128, s);
  const int ntiles = (q_end + 63) / 64;
  f32x16 dq[X::DT];
#pragma unroll
  for (int dt = 0; dt < X::DT; ++dt)
#pragma unroll
    for (int v = 0; v < 16; ++v) dq[dt][v] = 0.0f;
  const float sc = p.scale * LOG2E;
  const uint32_t smem_base = lds_addr(smem);

  issue_tile(0);
  for (int j = 0; j < ntiles; ++j) {
    if constexpr (D == 128) pin_acc(dq);
    wait_vmcnt<0>();
    __builtin_amdgcn_s_barrier();
    const int kv0 = j * 64;
    const bool hidden = kv0 > qw0 + 31;                       // every key of the tile is masked for this wave
    if constexpr (D == 128) {      // the other heads' tiles are asked for here, these between the tile's products: past the last one as well
      if (hidden) issue_tile(j + 1);
    } else {
      if (j + 1 < ntiles) issue_tile(j + 1);
    }
    if (hidden) continue;
    const uint32_t st = smem_base + (j & 1) * STAGE;
    const bool diagonal = kv0 + 63 > qw0;                   // the tile meets the diagonal
    if constexpr (D == 128) {
      f32x16 sT[2], dpT[2];
      uint32_t ds[2][8];
      auto powers = [&](auto tc, auto wc) {             // P^T of two keys of half T, in the place of their scores
        constexpr int T = decltype(tc)::value, W = decltype(wc)::value;
#pragma unroll
        for (int v = 2 * W; v < 2 * W + 2; ++v) sT[T][v] = exp2_raw(sT[T][v] * sc - lse2);
      };
      auto grads = [&](auto tc, auto wc) {              // dS^T, packed
        constexpr int T = decltype(tc)::value, W = decltype(wc)::value;
        ds[T][W] = pack_bf16(sT[T][2 * W] * (dpT[T][2 * W] - dq_dot), sT[T][2 * W + 1] * (dpT[T][2 * W + 1] - dq_dot));
      };
      // S^T = K Q^T and dP^T = V dO^T, then dQ^T += K^T dS^T
      bwd_tile<false>(st, st + RM_TILE, offP, offT, qf, dof, sT, dpT, [&] { start_scores(sT[0], diagonal, 0, qpos - kv0, fh); start_scores(sT[1], diagonal, 0, qpos - kv0 - 32, fh); },
                      [&](auto ic) {
                        constexpr int I = decltype(ic)::value;
                        ldr.issue_one(I % 4, I < 4 ? rsK : rsV, smem + ((j + 1) & 1) * STAGE + I / 4 * RM_TILE, (uint32_t)((j + 1) * 64) * (uint32_t)ld * 2u, wave);
                      },
                      [](auto) {}, powers, grads, [&](auto cc, auto&& use) {
                        constexpr int C = decltype(cc)::value;
                        if constexpr (std::is_same_v<std::decay_t<decltype(use)>, std::nullptr_t>) return st;
                        else use(ds[C], dq);
                      });
    } else {
      auto part = [&](bool masked, auto tc) {               // 32 keys at a time
        constexpr int T = decltype(tc)::value;
        f32x16 sT, dpT;
        start_scores(sT, masked, 0, qpos - kv0 - 32 * T, fh);
  #pragma unroll
        for (int v = 0; v < 16; ++v) dpT[v] = 0.0f;
        rm_mma_rows<D, T>(st, st + RM_TILE, offP, qf, dof, sT, dpT);      // S^T = K Q^T, dP^T = V dO^T
  #pragma unroll
        for (int v = 0; v < 16; ++v) sT[v] = exp2_raw(sT[v] * sc - lse2);
  #pragma unroll
        for (int v = 0; v < 16; ++v) sT[v] *= dpT[v] - dq_dot;
        bf16x8 dsf[2];
        pack_acc(sT, dsf);
        rm_mma_cols<D, T>(st, offT, dsf, dq);               // dQ^T += K^T dS^T
        __builtin_amdgcn_sched_barrier(0);
      };
      part(diagonal, half0{});
      part(diagonal, half1{});
    }
  }
  if constexpr (D == 128) { settle(dq); wait_vmcnt<0>(); }       // no load may land in the LDS once it is another workgroup's
  if (qpos < s) {
    bf16_t* out = static_cast<bf16_t*>(p.dqkv) + ((long)bi * s + qpos) * ld + hh * D;
    if (p.rope) rope_back<D>(dq, qpos, fh, p.rope_log2_base);
    store_transposed<D>(dq, p.scale, out, fh);
  }
}

// ------------------------------------------------------------------------------------- dK / dV pass
// P = exp(S - lse) into sm and dS = P (dP - D) into dpm for 32 queries: a lane's lse and D (256 bytes on) of group g of
// its rows lie in LDS at `stats` + 32 g bytes.
DEV void dkv_probs(uint32_t stats, float sc, f32x16& sm, f32x16& dpm) {
  u32x4 l4[4], d4[4];
  static_for<0, 4>([&](auto gc) {
    constexpr int G = decltype(gc)::value;
    l4[G] = ds_read_b128_at<32 * G>(stats);
    d4[G] = ds_read_b128_at<32 * G + 256>(stats);
  });
  lds_wait<0>();
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    tie(l4[g]);
    tie(d4[g]);
    const f32x4 lf = __builtin_bit_cast(f32x4, l4[g]), df = __builtin_bit_cast(f32x4, d4[g]);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      sm[4 * g + e] = exp2_raw(sm[4 * g + e] * sc - lf[e] * LOG2E);
      dpm[4 * g + e] -= df[e];
    }
  }
#pragma unroll
  for (int v = 0; v < 16; ++v) dpm[v] *= sm[v];
}

template <int D>
DEV void attn_bwd_dkv_body(const AttnArgs& p, uint8_t* smem, int kb, int hh, int bi) {
  using X = Dims<D>;
  constexpr int STAGE = 2 * RM_TILE + 512;                // Q tile, dO tile (64 queries), lse[64], dot[64]
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int fr = lane & 31, fh = lane >> 5;
  const int s = p.seq;                            // 128 keys per workgroup
  const int kw0 = kb * 128 + wave * 32, kpos = kw0 + fr;
  const long ld = p.ld, ldc = p.ld_ctx;
  const bf16_t* tok0 = static_cast<const bf16_t*>(p.qkv) + (long)bi * s * ld;
  const bf16_t* do0 = static_cast<const bf16_t*>(p.dctx) + (long)bi * s * ldc + hh * D;
  const int hl = p.heads * D;
  const buf_rsrc rsQ = make_rsrc(tok0 + hh * D, ((long)(s - 1) * ld + D) * 2);
  const buf_rsrc rsO = make_rsrc(do0, ((long)(s - 1) * ldc + D) * 2);
  const long stat0 = ((long)bi * p.heads + hh) * s;
  const buf_rsrc rsL = make_rsrc(p.lse + stat0, (long)s * 4);   // rows past the end read as 0: harmless, their
  const buf_rsrc rsD = make_rsrc(p.dot + stat0, (long)s * 4);   // Q and dO rows are zero as well

  bf16x8 kf[X::KSTEPS], vf[X::KSTEPS];
  load_row_frags<D>(tok0 + hl + hh * D, ld, kpos, s, fh, kf);
  load_row_frags<D>(tok0 + 2 * hl + hh * D, ld, kpos, s, fh, vf);
  if constexpr (D == 128) { keep_in_acc(kf); keep_in_acc(vf); }

  RmLoader ldq, ldo;
  ldq.init((int)ld, D, wave, lane);
  ldo.init((int)ldc, D, wave, lane);
  auto issue_stats = [&](int j, uint8_t* st) {
    if (wave == 0) __builtin_amdgcn_raw_ptr_buffer_load_lds(rsL, LDS_PTR(st + 2 * RM_TILE), 4, (uint32_t)(j * 64 + lane) * 4u, 0, 0, 0);
    if (wave == 1) __builtin_amdgcn_raw_ptr_buffer_load_lds(rsD, LDS_PTR(st + 2 * RM_TILE + 256), 4, (uint32_t)(j * 64 + lane) * 4u, 0, 0, 0);
  };
  auto issue_tile = [&](int j, int slot) {
    uint8_t* st = smem + slot * STAGE;
    ldq.issue(rsQ, st, (uint32_t)(j * 64) * (uint32_t)ld * 2u, wave);
    ldo.issue(rsO, st + RM_TILE, (uint32_t)(j * 64) * (uint32_t)ldc * 2u, wave);
    issue_stats(j, st);
  };
  const uint32_t offP = rm_plain_off(lane), offT = rm_trans_off(lane);

  const int nq = (s + 63) / 64;
  const int j0 = (kb * 128) / 64;                         // first query tile that sees these keys
  f32x16 dk[X::DT], dv[X::DT];
#pragma unroll
  for (int dt = 0; dt < X::DT; ++dt)
#pragma unroll
    for (int v = 0; v < 16; ++v) { dk[dt][v] = 0.0f; dv[dt][v] = 0.0f; }
  const float sc = p.scale * LOG2E;
  const uint32_t smem_base = lds_addr(smem);

  issue_tile(j0, 0);
  for (int j = j0; j < nq; ++j) {
    if constexpr (D == 128) { pin_acc(dk); pin_acc(dv); }
    const int slot = (j - j0) & 1;
    wait_vmcnt<0>();
    __builtin_amdgcn_s_barrier();
    const int q0 = j * 64;
    const bool hidden = q0 + 63 < kw0;                    // no query of the tile sees this wave's keys
    if constexpr (D == 128) {      // as in the dQ pass
      if (hidden) issue_tile(j + 1, slot ^ 1); else issue_stats(j + 1, smem + (slot ^ 1) * STAGE);
    } else {
      if (j + 1 < nq) issue_tile(j + 1, slot ^ 1);
    }
    if (hidden) continue;
    const uint32_t st = smem_base + slot * STAGE;
    const bool diagonal = q0 < kw0 + 31;                    // the tile meets the diagonal
    if constexpr (D == 128) {
      f32x16 sm[2], dpm[2];
      uint32_t pw[2][8], ds[2][8];
      u32x4 l4[4], d4[4];
      auto read_stats = [&](auto ic) {                  // lse and D of four of the lane's queries (half 0, then half 1)
        constexpr int T = decltype(ic)::value / 4, G = decltype(ic)::value % 4;
        l4[G] = ds_read_b128_at<2 * RM_TILE + 128 * T + 32 * G>(st + 16 * fh);
        d4[G] = ds_read_b128_at<2 * RM_TILE + 128 * T + 32 * G + 256>(st + 16 * fh);
      };
      auto powers = [&](auto tc, auto wc) {             // P of two queries of half T, in the place of their scores
        constexpr int T = decltype(tc)::value, W = decltype(wc)::value, G = W / 2;
        if constexpr (W % 2 == 0) asm volatile("" : "+v"(l4[G]), "+v"(d4[G]));       // behind the wait of this step
        const f32x4 lf = __builtin_bit_cast(f32x4, l4[G]);
#pragma unroll
        for (int v = 2 * W; v < 2 * W + 2; ++v) sm[T][v] = exp2_raw(sm[T][v] * sc - lf[v & 3] * LOG2E);
      };
      auto grads = [&](auto tc, auto wc) {              // P and dS, packed
        constexpr int T = decltype(tc)::value, W = decltype(wc)::value, V = 2 * W;
        const f32x4 df = __builtin_bit_cast(f32x4, d4[W / 2]);
        pw[T][W] = pack_bf16(sm[T][V], sm[T][V + 1]);
        ds[T][W] = pack_bf16(sm[T][V] * (dpm[T][V] - df[V & 3]), sm[T][V + 1] * (dpm[T][V + 1] - df[(V + 1) & 3]));
      };
      // S[q, kv] = Q K^T and dP[q, kv] = dO V^T, then dV^T += dO^T P and dK^T += Q^T dS
      bwd_tile<true>(st, st + RM_TILE, offP, offT, kf, vf, sm, dpm, [&] { start_scores(sm[0], diagonal, kpos - q0, 31, fh); start_scores(sm[1], diagonal, kpos - q0 - 32, 31, fh); },
                     [&](auto ic) {
                       constexpr int I = decltype(ic)::value;
                       uint8_t* next = smem + (slot ^ 1) * STAGE;
                       if constexpr (I < 4) ldq.issue_one(I, rsQ, next, (uint32_t)((j + 1) * 64) * (uint32_t)ld * 2u, wave);
                       else ldo.issue_one(I - 4, rsO, next + RM_TILE, (uint32_t)((j + 1) * 64) * (uint32_t)ldc * 2u, wave);
                     },
                     read_stats, powers, grads, [&](auto cc, auto&& use) {
                       constexpr int C = decltype(cc)::value;
                       if constexpr (std::is_same_v<std::decay_t<decltype(use)>, std::nullptr_t>) return C % 2 == 0 ? st + RM_TILE : st;
                       else if constexpr (C % 2 == 0) use(pw[C / 2], dv);
                       else use(ds[C / 2], dk);
                     });
    } else {
      auto part = [&](bool masked, auto tc) {               // 32 queries at a time
        constexpr int T = decltype(tc)::value;
        f32x16 sm, dpm;
        start_scores(sm, masked, kpos - q0 - 32 * T, 31, fh);
  #pragma unroll
        for (int v = 0; v < 16; ++v) dpm[v] = 0.0f;
        rm_mma_rows<D, T>(st, st + RM_TILE, offP, kf, vf, sm, dpm);       // S[q, kv] = Q K^T, dP[q, kv] = dO V^T
        dkv_probs(st + 2 * RM_TILE + (uint32_t)(32 * T + 4 * fh) * 4u, sc, sm, dpm);
        bf16x8 pf[2], dsf[2];
        pack_acc(sm, pf);
        pack_acc(dpm, dsf);
        rm_mma_cols<D, T>(st + RM_TILE, offT, pf, dv);      // dV^T += dO^T P
        rm_mma_cols<D, T>(st, offT, dsf, dk);               // dK^T += Q^T dS
        __builtin_amdgcn_sched_barrier(0);
      };
      part(diagonal, half0{});
      part(diagonal, half1{});
    }
  }
  if constexpr (D == 128) { settle(dk); settle(dv); wait_vmcnt<0>(); }
  if (kpos < s) {
    bf16_t* out = static_cast<bf16_t*>(p.dqkv) + ((long)bi * s + kpos) * ld + hh * D;
    if (p.rope) rope_back<D>(dk, kpos, fh, p.rope_log2_base);
    store_transposed<D>(dk, p.scale, out + hl, fh);
    store_transposed<D>(dv, 1.0f, out + 2 * hl, fh);
  }
}


// Both backward passes in one launch (they are independent given D, so one launch puts twice as many
// workgroups on the chip and the attention backward leaves its slice's critical path sooner).  Inside a
// (batch, head) group the items alternate, longest first: dK/dV pass of key block 0, dQ pass of the last query
// block, dK/dV pass of key block 1, ...
template <int D>
__global__ __launch_bounds__(256, D == 128 ? 1 : 2)
void attn_bwd_kernel(const AttnArgs p) {
  extern __shared__ __align__(1024) uint8_t smem[];
  const int nxb = (p.seq + 127) / 128;
  int pos, group;
  if (!ranked_item(2 * nxb, p.heads * p.batch, pos, group)) return;
  const int hh = group % p.heads, bi = group / p.heads;
  if (pos & 1) attn_bwd_dq_body<D>(p, smem, nxb - 1 - (pos >> 1), hh, bi);
  else attn_bwd_dkv_body<D>(p, smem, pos >> 1, hh, bi);
}


// ------------------------------------------------------------------------------------- few workgroups
// With few (batch element, head) pairs or short sequences the passes above are one serial chain per workgroup (64 keys
// or queries a step, 1.2 us forward and 1.6 us backward with heads of 128) on a chip that is mostly idle.  Here a workgroup
// owns 32 queries (keys), and its four waves deal the other side's 32-row tiles among themselves: four times the
// workgroups, a quarter of the chain.  Every wave stages its own tiles (no barrier inside the loop), and the waves' sums
// meet in LDS at the end, added in wave order.
constexpr int SP_TILE = 8192;                    // 32 positions of a row-major tile
constexpr int SP_STAGE = 2 * SP_TILE + 512;      // two tiles, and lse[64], dot[64] where a pass needs them
constexpr int SP_WAVE = 2 * SP_STAGE;            // a wave's LDS: two stages, its sums afterwards

struct SplitLoader {         // one wave, 8 one-KiB pieces (4 rows each) of a 32-row tile
  uint32_t base[8];
  DEV void init(int ld, int d_valid, int lane) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int row = 4 * i + (lane >> 4);
      const int d = ((lane & 15) ^ rm_swz(row)) * 8;
      base[i] = d < d_valid ? (uint32_t)(row * ld + d) * 2u : BUF_OOB;
    }
  }
  DEV void issue(buf_rsrc rs, uint8_t* tile, uint32_t row_byte_off) const {
#pragma unroll
    for (int i = 0; i < 8; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, LDS_PTR(tile + i * 1024), 16, base[i] + row_byte_off, 0, 0, 0);
  }
};

// Accumulators to LDS and back, 16 bytes a lane: value group (dt, g) of lane l at ((4 dt + g) * 64 + l) * 16.
template <int N>
DEV void put_acc(uint8_t* at, const f32x16 (&o)[N], int lane) {
#pragma unroll
  for (int dt = 0; dt < N; ++dt)
#pragma unroll
    for (int g = 0; g < 4; ++g)
      *reinterpret_cast<f32x4*>(at + ((4 * dt + g) * 64 + lane) * 16) = f32x4{o[dt][4 * g], o[dt][4 * g + 1], o[dt][4 * g + 2], o[dt][4 * g + 3]};
}
template <int N>
DEV void sum_acc(const uint8_t* at, f32x16 (&o)[N], int lane) {      // over the four waves, in wave order
#pragma unroll
  for (int dt = 0; dt < N; ++dt)
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      f32x4 v = *reinterpret_cast<const f32x4*>(at + ((4 * dt + g) * 64 + lane) * 16);
#pragma unroll
      for (int w = 1; w < 4; ++w) v += *reinterpret_cast<const f32x4*>(at + w * SP_WAVE + ((4 * dt + g) * 64 + lane) * 16);
#pragma unroll
      for (int e = 0; e < 4; ++e) o[dt][4 * g + e] = v[e];
    }
}
template <int D>
DEV void zero_acc(f32x16 (&o)[Dims<D>::DT]) {
#pragma unroll
  for (int dt = 0; dt < Dims<D>::DT; ++dt)
#pragma unroll
    for (int v = 0; v < 16; ++v) o[dt][v] = 0.0f;
}

template <int D>
__global__ __launch_bounds__(256)
void attn_fwd_split_kernel(const AttnArgs p) {
  using X = Dims<D>;
  extern __shared__ __align__(1024) uint8_t smem[];
  __shared__ float stat_m[4][64], stat_l[4][64];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int fr = lane & 31, fh = lane >> 5;
  const int s = p.seq, nqb = (s + 31) / 32;
  int pos, group;
  if (!ranked_item(nqb, p.heads * p.batch, pos, group)) return;
  const int qb = nqb - 1 - pos, hh = group % p.heads, bi = group / p.heads;
  const int qpos = qb * 32 + fr;
  const long ld = p.ld;
  const bf16_t* tok0 = static_cast<const bf16_t*>(p.qkv) + (long)bi * s * ld;
  const int hl = p.heads * D;
  const long view_bytes = ((long)(s - 1) * ld + D) * 2;
  const buf_rsrc rsK = make_rsrc(tok0 + hl + hh * D, view_bytes);
  const buf_rsrc rsV = make_rsrc(tok0 + 2 * hl + hh * D, view_bytes);
  uint8_t* const mine = smem + wave * SP_WAVE;
  SplitLoader ldr;
  ldr.init((int)ld, D, lane);
  auto issue = [&](int j, int stage) {
    const uint32_t ro = (uint32_t)(j * 32) * (uint32_t)ld * 2u;
    ldr.issue(rsK, mine + stage * SP_STAGE, ro);
    ldr.issue(rsV, mine + stage * SP_STAGE + SP_TILE, ro);
  };
  if (wave <= qb) issue(wave, 0);
  bf16x8 qf[X::KSTEPS];
  load_row_frags<D>(tok0 + hh * D, ld, qpos, s, fh, qf);
  const uint32_t offP = rm_plain_off(lane), offT = rm_trans_off(lane);
  f32x16 o[X::DT];
  zero_acc<D>(o);
  float m = -INFINITY, l = 0.0f;
  const float sc = p.scale * LOG2E;
  int stage = 0;
  for (int j = wave; j <= qb; j += 4, stage ^= 1) {
    if (j + 4 <= qb) { issue(j + 4, stage ^ 1); wait_vmcnt<16>(); } else { wait_vmcnt<0>(); }
    const uint32_t st = lds_addr(mine) + stage * SP_STAGE;
    f32x16 sT;
    start_scores(sT, j == qb, 0, qpos - j * 32, fh);
    u32x4 kf[X::KSTEPS];
    static_for<0, X::KSTEPS>([&](auto kc) { constexpr int K = decltype(kc)::value; kf[K] = ds_read_b128_at<0>(st + (offP ^ (K << 5))); });
    u32x2 vf[2][2][2];
    auto read_v = [&](auto dd) {
      constexpr int DTI = decltype(dd)::value;
      static_for<0, 2>([&](auto uu) {
        constexpr int U = decltype(uu)::value;
        vf[DTI & 1][U][0] = ds_read_tr_at<SP_TILE + U * 4096>(st + (offT ^ ((4 * DTI) << 4)));
        vf[DTI & 1][U][1] = ds_read_tr_at<SP_TILE + U * 4096 + 2048>(st + (offT ^ (((4 * DTI) ^ 2) << 4)));
      });
    };
    lds_wait<0>();
#pragma unroll
    for (int k = 0; k < X::KSTEPS; ++k) {
      tie(kf[k]);
      sT = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kf[k]), qf[k], sT, 0, 0, 0);     // S^T[kv, q] = K Q^T
    }
    float mx = -INFINITY;
#pragma unroll
    for (int v = 0; v < 16; ++v) mx = fmaxf(mx, sT[v]);
    mx = fmaxf(mx, other_half(mx)) * sc;
    const float m_new = fmaxf(m, mx);                    // finite: the first key of any tile up to the diagonal is visible
    if (__builtin_amdgcn_ballot_w64(m_new != m) != 0) {
      const float alpha = exp2_raw(m - m_new);
      l *= alpha;
#pragma unroll
      for (int dt = 0; dt < X::DT; ++dt)
#pragma unroll
        for (int v = 0; v < 16; ++v) o[dt][v] *= alpha;
      m = m_new;
    }
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      sT[v] = exp2_raw(sT[v] * sc - m);
      l += sT[v];
    }
    bf16x8 pf[2];
    pack_acc(sT, pf);
    read_v(std::integral_constant<int, 0>{});
    static_for<0, X::DT>([&](auto dd) {                  // O^T[d, q] += V^T P^T
      constexpr int DTI = decltype(dd)::value;
      if constexpr (DTI + 1 < X::DT) read_v(std::integral_constant<int, DTI + 1>{});
      lds_wait<(DTI + 1 < X::DT) ? 4 : 0>();
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        tie(vf[DTI & 1][u][0]);
        tie(vf[DTI & 1][u][1]);
        const u32x4 a = {vf[DTI & 1][u][0][0], vf[DTI & 1][u][0][1], vf[DTI & 1][u][1][0], vf[DTI & 1][u][1][1]};
        o[DTI] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), pf[u], o[DTI], 0, 0, 0);
      }
    });
  }
  l += other_half(l);
  stat_m[wave][lane] = m;
  stat_l[wave][lane] = l;
  __syncthreads();
  float m_all = -INFINITY, l_all = 0.0f;
#pragma unroll
  for (int w = 0; w < 4; ++w) m_all = fmaxf(m_all, stat_m[w][lane]);
#pragma unroll
  for (int w = 0; w < 4; ++w) l_all += stat_l[w][lane] * exp2_raw(stat_m[w][lane] - m_all);     // a wave without a tile: 2^-inf = 0
  const float mine_scale = exp2_raw(m - m_all);
#pragma unroll
  for (int dt = 0; dt < X::DT; ++dt)
#pragma unroll
    for (int v = 0; v < 16; ++v) o[dt][v] *= mine_scale;
  put_acc(mine, o, lane);
  __syncthreads();
  if (wave == 0) {
    sum_acc(smem, o, lane);
    if (qpos < s) {
      bf16_t* out = static_cast<bf16_t*>(p.ctx) + ((long)bi * s + qpos) * p.ld_ctx + hh * D;
      store_transposed<D>(o, 1.0f / l_all, out, fh);
      if (fh == 0) p.lse[((long)bi * p.heads + hh) * s + qpos] = (m_all + log2f(l_all)) * LN2;
    }
  }
}

// D = rowsum(dO * O) of 32 queries is the diagonal of dO O^T: with OWN_D the passes form it by the MFMAs that form dP, in the same order.
// See attention_owns_d for where that pays.
// Lane c, or the one 32 on, holds the diagonal's value c: lanes whose half is diag_half(c).
DEV int diag_half(int c) { return (c >> 2) & 1; }
DEV float diag(const f32x16& t, int c) {
  float d = t[0];
#pragma unroll
  for (int v = 1; v < 16; ++v) d = 4 * (c >> 3) + (c & 3) == v ? t[v] : d;
  return d;
}

template <int D, bool OWN_D>
DEV void attn_bwd_dq_split_body(const AttnArgs& p, uint8_t* smem, int qb, int hh, int bi) {
  using X = Dims<D>;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int fr = lane & 31, fh = lane >> 5;
  const int s = p.seq, qpos = qb * 32 + fr;
  const long ld = p.ld;
  const bf16_t* tok0 = static_cast<const bf16_t*>(p.qkv) + (long)bi * s * ld;
  const int hl = p.heads * D;
  const long view_bytes = ((long)(s - 1) * ld + D) * 2;
  const buf_rsrc rsK = make_rsrc(tok0 + hl + hh * D, view_bytes);
  const buf_rsrc rsV = make_rsrc(tok0 + 2 * hl + hh * D, view_bytes);
  uint8_t* const mine = smem + wave * SP_WAVE;
  SplitLoader ldr;
  ldr.init((int)ld, D, lane);
  auto issue = [&](int j, int stage) {
    const uint32_t ro = (uint32_t)(j * 32) * (uint32_t)ld * 2u;
    ldr.issue(rsK, mine + stage * SP_STAGE, ro);
    ldr.issue(rsV, mine + stage * SP_STAGE + SP_TILE, ro);
  };
  if (wave <= qb) issue(wave, 0);
  bf16x8 qf[X::KSTEPS], dof[X::KSTEPS];
  load_row_frags<D>(tok0 + hh * D, ld, qpos, s, fh, qf);
  load_row_frags<D>(static_cast<const bf16_t*>(p.dctx) + (long)bi * s * p.ld_ctx + hh * D, p.ld_ctx, qpos, s, fh, dof);
  const long stat = ((long)bi * p.heads + hh) * s + qpos;
  const float lse2 = qpos < s ? p.lse[stat] * LOG2E : INFINITY;
  float dq_dot;
  if constexpr (!OWN_D) {
    dq_dot = qpos < s ? p.dot[stat] : 0.0f;
  } else {
    bf16x8 of[X::KSTEPS];
    load_row_frags<D>(static_cast<const bf16_t*>(p.ctx) + (long)bi * s * p.ld_ctx + hh * D, p.ld_ctx, qpos, s, fh, of);
    f32x16 sums;
#pragma unroll
    for (int v = 0; v < 16; ++v) sums[v] = 0.0f;
#pragma unroll
    for (int k = 0; k < X::KSTEPS; ++k) sums = __builtin_amdgcn_mfma_f32_32x32x16_bf16(of[k], dof[k], sums, 0, 0, 0);
    const float mine_d = diag(sums, fr), other_d = other_half(mine_d);
    dq_dot = fh == diag_half(fr) ? mine_d : other_d;
  }
  const uint32_t offP = rm_plain_off(lane), offT = rm_trans_off(lane);
  const float sc = p.scale * LOG2E;
  f32x16 dq[X::DT];
  zero_acc<D>(dq);
  int stage = 0;
  for (int j = wave; j <= qb; j += 4, stage ^= 1) {
    if (j + 4 <= qb) { issue(j + 4, stage ^ 1); wait_vmcnt<16>(); } else { wait_vmcnt<0>(); }
    const uint32_t st = lds_addr(mine) + stage * SP_STAGE;
    {
      f32x16 sT, dpT;
      start_scores(sT, j == qb, 0, qpos - j * 32, fh);
#pragma unroll
      for (int v = 0; v < 16; ++v) dpT[v] = 0.0f;
      rm_mma_rows<D, 0>(st, st + SP_TILE, offP, qf, dof, sT, dpT);
#pragma unroll
      for (int v = 0; v < 16; ++v) sT[v] = exp2_raw(sT[v] * sc - lse2);
#pragma unroll
      for (int v = 0; v < 16; ++v) sT[v] *= dpT[v] - dq_dot;
      bf16x8 dsf[2];
      pack_acc(sT, dsf);
      rm_mma_cols<D, 0>(st, offT, dsf, dq);
    }
  }
  put_acc(mine, dq, lane);
  __syncthreads();
  if (wave == 0 && qpos < s) {
    sum_acc(smem, dq, lane);
    bf16_t* out = static_cast<bf16_t*>(p.dqkv) + ((long)bi * s + qpos) * ld + hh * D;
    if (p.rope) rope_back<D>(dq, qpos, fh, p.rope_log2_base);
    store_transposed<D>(dq, p.scale, out, fh);
  }
}

template <int D, bool OWN_D>
DEV void attn_bwd_dkv_split_body(const AttnArgs& p, uint8_t* smem, int kb, int hh, int bi) {
  using X = Dims<D>;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int fr = lane & 31, fh = lane >> 5;
  const int s = p.seq, kpos = kb * 32 + fr, nq = (s + 31) / 32;
  const long ld = p.ld, ldc = p.ld_ctx;
  const bf16_t* tok0 = static_cast<const bf16_t*>(p.qkv) + (long)bi * s * ld;
  const bf16_t* do0 = static_cast<const bf16_t*>(p.dctx) + (long)bi * s * ldc + hh * D;
  const int hl = p.heads * D;
  const buf_rsrc rsQ = make_rsrc(tok0 + hh * D, ((long)(s - 1) * ld + D) * 2);
  const buf_rsrc rsO = make_rsrc(do0, ((long)(s - 1) * ldc + D) * 2);
  const long stat0 = ((long)bi * p.heads + hh) * s;
  const buf_rsrc rsL = make_rsrc(p.lse + stat0, (long)s * 4);
  const buf_rsrc rsD = make_rsrc(p.dot + stat0, (long)s * 4);
  const buf_rsrc rsC = make_rsrc(static_cast<const bf16_t*>(p.ctx) + (long)bi * s * ldc + hh * D, ((long)(s - 1) * ldc + D) * 2);
  uint8_t* const mine = smem + wave * SP_WAVE;
  SplitLoader ldq, ldo;
  ldq.init((int)ld, D, lane);
  ldo.init((int)ldc, D, lane);
  auto issue = [&](int j, int stage) {
    uint8_t* st = mine + stage * SP_STAGE;
    ldq.issue(rsQ, st, (uint32_t)(j * 32) * (uint32_t)ld * 2u);
    ldo.issue(rsO, st + SP_TILE, (uint32_t)(j * 32) * (uint32_t)ldc * 2u);
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rsL, LDS_PTR(st + 2 * SP_TILE), 4, (uint32_t)(j * 32 + lane) * 4u, 0, 0, 0);
    if constexpr (!OWN_D) __builtin_amdgcn_raw_ptr_buffer_load_lds(rsD, LDS_PTR(st + 2 * SP_TILE + 256), 4, (uint32_t)(j * 32 + lane) * 4u, 0, 0, 0);
  };
  const uint32_t o_off = (uint32_t)(fr * (int)ldc + fh * 8) * 2u;
  if (kb + wave < nq) issue(kb + wave, 0);
  bf16x8 kf[X::KSTEPS], vf[X::KSTEPS];
  load_row_frags<D>(tok0 + hl + hh * D, ld, kpos, s, fh, kf);
  load_row_frags<D>(tok0 + 2 * hl + hh * D, ld, kpos, s, fh, vf);
  const uint32_t offP = rm_plain_off(lane), offT = rm_trans_off(lane);
  const float sc = p.scale * LOG2E;
  f32x16 dk[X::DT], dv[X::DT];
  zero_acc<D>(dk);
  zero_acc<D>(dv);
  int stage = 0;
  for (int j = kb + wave; j < nq; j += 4, stage ^= 1) {
    // O of this tile straight into fragments, asked for in front of the next tile so that it can be waited for alone, and needed
    // behind the scores
    u32x4 of[OWN_D ? X::KSTEPS : 1];
    if constexpr (OWN_D) {
#pragma unroll
      for (int k = 0; k < X::KSTEPS; ++k) of[k] = __builtin_amdgcn_raw_buffer_load_b128(rsC, o_off + (uint32_t)(j * 32) * (uint32_t)ldc * 2u + 32u * k, 0, 0);
      issue(j + 4, stage ^ 1);                             // past the last one too: zeros, and one count of loads for the compiler's waits
      asm volatile("" ::: "memory");                       // none of them is moved behind the wait
      __builtin_amdgcn_sched_barrier(0);
      wait_vmcnt<X::KSTEPS + 17>();
    } else if (j + 4 < nq) {
      issue(j + 4, stage ^ 1);
      wait_vmcnt<18>();
    } else {
      wait_vmcnt<0>();
    }
    const uint32_t st = lds_addr(mine) + stage * SP_STAGE;
    {
      f32x16 sm, dpm;
      start_scores(sm, j == kb, kpos - j * 32, 31, fh);
#pragma unroll
      for (int v = 0; v < 16; ++v) dpm[v] = 0.0f;
      rm_mma_rows<D, 0>(st, st + SP_TILE, offP, kf, vf, sm, dpm);
      if constexpr (OWN_D) {
        f32x16 sums;                                         // dO O^T, its diagonal to where D is read from
#pragma unroll
        for (int v = 0; v < 16; ++v) sums[v] = 0.0f;
        u32x4 dof[X::KSTEPS];
        static_for<0, X::KSTEPS>([&](auto kc) { constexpr int K = decltype(kc)::value; dof[K] = ds_read_b128_at<SP_TILE>(st + (offP ^ (K << 5))); });
        lds_wait<0>();
#pragma unroll
        for (int k = 0; k < X::KSTEPS; ++k) {
          tie(dof[k]);
          sums = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, dof[k]), __builtin_bit_cast(bf16x8, of[k]), sums, 0, 0, 0);
        }
        const float d = diag(sums, fr);
        if (fh == diag_half(fr)) asm volatile("ds_write_b32 %0, %1 offset:%2" ::"v"(st + 4u * fr), "v"(d), "n"(2 * SP_TILE + 256) : "memory");
      }
      dkv_probs(st + 2 * SP_TILE + (uint32_t)fh * 16u, sc, sm, dpm);
      bf16x8 pf[2], dsf[2];
      pack_acc(sm, pf);
      pack_acc(dpm, dsf);
      rm_mma_cols<D, 0>(st + SP_TILE, offT, pf, dv);
      rm_mma_cols<D, 0>(st, offT, dsf, dk);
    }
  }
  if constexpr (OWN_D) wait_vmcnt<0>();                    // no load may land in what the sums go to
  put_acc(mine, dk, lane);
  put_acc(mine + X::DT * 4096, dv, lane);
  __syncthreads();
  if (kpos >= s) return;
  bf16_t* out = static_cast<bf16_t*>(p.dqkv) + ((long)bi * s + kpos) * ld + hh * D;
  if (wave == 0) {
    sum_acc(smem, dk, lane);
    if (p.rope) rope_back<D>(dk, kpos, fh, p.rope_log2_base);
    store_transposed<D>(dk, p.scale, out + hl, fh);
  } else if (wave == 1) {
    sum_acc(smem + X::DT * 4096, dv, lane);
    store_transposed<D>(dv, 1.0f, out + 2 * hl, fh);
  }
}

template <int D, bool OWN_D>
__global__ __launch_bounds__(256)
void attn_bwd_split_kernel(const AttnArgs p) {
  static_assert(SP_WAVE >= 2 * Dims<D>::DT * 4096, "a wave's dK and dV sums fit its stages");
  extern __shared__ __align__(1024) uint8_t smem[];
  const int nb = (p.seq + 31) / 32;
  int pos, group;
  if (!ranked_item(2 * nb, p.heads * p.batch, pos, group)) return;
  const int hh = group % p.heads, bi = group / p.heads;
  if (pos & 1) attn_bwd_dq_split_body<D, OWN_D>(p, smem, nb - 1 - (pos >> 1), hh, bi);
  else attn_bwd_dkv_split_body<D, OWN_D>(p, smem, pos >> 1, hh, bi);
}

template <int D>
hipError_t fwd_launch(const AttnArgs& a, hipStream_t st) {
  if (attention_split_pays(a, false)) {
    constexpr int LDS = 4 * SP_WAVE;
    static LdsLimitOnce lds_limit;
    hipError_t e = lds_limit.ensure(reinterpret_cast<const void*>(attn_fwd_split_kernel<D>), LDS);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(attn_fwd_split_kernel<D>, dim3(ranked_grid((a.seq + 31) / 32, a.heads * a.batch)), dim3(256), LDS, st, a);
    return hipGetLastError();
  }
  constexpr int LDS = 2 * (((D + 31) / 32) * 4096 + 2 * 8192);      // both forms
  const dim3 grid(ranked_grid((a.seq + 127) / 128, a.heads * a.batch));
  if (attention_fwd_serial(a)) {
    static LdsLimitOnce lds_limit;
    if (hipError_t e = lds_limit.ensure(reinterpret_cast<const void*>(attn_fwd_serial_kernel<D>), LDS); e != hipSuccess) return e;
    hipLaunchKernelGGL(attn_fwd_serial_kernel<D>, grid, dim3(256), LDS, st, a);
    return hipGetLastError();
  }
  static LdsLimitOnce lds_limit;
  if (hipError_t e = lds_limit.ensure(reinterpret_cast<const void*>(attn_fwd_kernel<D>), LDS); e != hipSuccess) return e;
  hipLaunchKernelGGL(attn_fwd_kernel<D>, grid, dim3(256), LDS, st, a);
  return hipGetLastError();
}

template <int D, bool OWN_D>
hipError_t bwd_split_launch(const AttnArgs& a, hipStream_t st) {
  constexpr int LDS = 4 * SP_WAVE;
  static LdsLimitOnce lds_limit;
  if (hipError_t e = lds_limit.ensure(reinterpret_cast<const void*>(attn_bwd_split_kernel<D, OWN_D>), LDS); e != hipSuccess) return e;
  hipLaunchKernelGGL((attn_bwd_split_kernel<D, OWN_D>), dim3(ranked_grid(2 * ((a.seq + 31) / 32), a.heads * a.batch)), dim3(256), LDS, st, a);
  return hipGetLastError();
}

template <int D>
hipError_t bwd_launch(const AttnArgs& a, hipStream_t st) {
  const bool split = attention_split_pays(a, true);
  if (split && attention_owns_d(a.seq)) return bwd_split_launch<D, true>(a, st);
  const int rows = a.batch * a.seq;
  hipLaunchKernelGGL(attn_dot_kernel<D>, dim3((unsigned)(((long)rows * a.heads + 63) / 64)), dim3(64), 0, st,
                     static_cast<const bf16_t*>(a.ctx), static_cast<const bf16_t*>(a.dctx), a.ld_ctx, rows, a.seq, a.heads, a.dot);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (split) return bwd_split_launch<D, false>(a, st);
  constexpr int LDS = 2 * (2 * RM_TILE + 512);             // the larger of the two passes' needs
  static LdsLimitOnce lds_limit;
  if ((e = lds_limit.ensure(reinterpret_cast<const void*>(attn_bwd_kernel<D>), LDS)) != hipSuccess) return e;
  const dim3 grid(ranked_grid(2 * ((a.seq + 127) / 128), a.heads * a.batch));
  hipLaunchKernelGGL(attn_bwd_kernel<D>, grid, dim3(256), LDS, st, a);
  return hipGetLastError();
}

}  // namespace

hipError_t attention_fwd_launch(const AttnArgs& a, hipStream_t st) {
  switch (a.head_dim) {
    case 64: return fwd_launch<64>(a, st);
    case 80: return fwd_launch<80>(a, st);
    case 128: return fwd_launch<128>(a, st);
    default: return hipErrorInvalidValue;
  }
}

hipError_t attention_bwd_launch(const AttnArgs& a, hipStream_t st) {
  switch (a.head_dim) {
    case 64: return bwd_launch<64>(a, st);
    case 80: return bwd_launch<80>(a, st);
    case 128: return bwd_launch<128>(a, st);
    default: return hipErrorInvalidValue;
  }
}
