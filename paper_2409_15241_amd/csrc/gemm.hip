// bf16 MFMA GEMM for gfx950 with fused epilogues: the products of Eq. 1-4 (X*A, (XA)*B_j) and the
// two products of every "grad matmul" (Sec. 4.1.2: input gradient and weight gradient).
//
//   C[m][n] = epilogue( sum_k Aop(m,k) * Bop(k,n) ),  fp32 accumulation in MFMA 16x16x32.
//
// Each operand is either contraction-contiguous in memory (KC: [row][k]) or contraction-strided
// (KS: [k][row]); see lds_dma.h.  The three products of a linear layer map to
//   forward   X[M,K]   * W[K,N]            : A KC, B KS
//   dgrad     dY[M,N'] * W[K',N']^T        : A KC, B KC   (contraction over N')
//   wgrad     X[M',K']^T * dY[M',N]        : A KS, B KS   (contraction over the tokens M')
//
// Work decomposition: one workgroup of four waves (one per SIMD) per BM x BN tile of C, each wave owning a
// WM x WN sub-tile as (WN/16) x (WM/16) MFMA accumulators.  Operand tiles of BK = 64 contraction elements (whole
// 128-byte lines of a contraction-contiguous operand) travel HBM/L2 -> LDS with buffer_load ... lds into two rings
// (see Rings); no VGPR staging, no ds_write.
// What bounds it at large sizes is power: a 16x16x32 MFMA reads and writes half as many accumulator bytes per flop as
// a 32x32x16 one (1.89 against 1.83 PFLOP/s at 0.545 against 0.549 pJ/flop above idle on N(0,1) x N(0,0.02) fragments with
// nothing else running, which domino_mfma_probe_shape measures), so every product here is made of those; a wave tile of
// 128x128 reads 64 bytes of fragments per clock and compute unit at full rate where 128x64 reads 96.  All whole-tile forms
// sum the contraction in the same order (32 elements per MFMA), so the bits do not depend on the tile shape; the dealt
// forms (gemm_split_body) sum it per wave.
// The MFMA is issued with the roles swapped (first operand = B fragment) so that a lane ends up
// with 4 consecutive n for one m: 8-byte bf16 / 16-byte fp32 stores.
#include "gemm.h"
#include "host_once.h"
#include "lds_dma.h"
#include "norm_body.h"
#include <type_traits>

namespace {

constexpr int BK = GEMM_BK;
// Operand tiles in LDS at once, of A and of B (see the software pipeline of gemm_body).  Weights come from HBM, the activations
// often from a cache that the kernel before has just written, and a place more is half to one and a half tiles more to
// land in: 256x128 tiles work through theirs in 0.6 us, so along a deep contraction they take all 160 KB, and in 192x256 the third place
// is B's, the larger tile of the two.  (A just written, B out of the caches, {3, 2} and as here: 2048 x 2560 x 5120 in 256x128 NN 70 -> 66 us,
// NT 74 -> 69, 3000 x 2000 x 2560 NN 37.6 -> 35.9, in 192x256 103 -> 92 and 97 -> 87, 2048 x 5120 x 2560 51.5 -> 48.2.  256x256 with {2, 3}
// and five places of each in 128x128 tiles, one workgroup to a compute unit, won here and lost there.)  DEEP: a third tile of both in front
// of the loop costs every 256x128 tile 0.2 to 0.5 us, which a shallow contraction does not win back (ring_pays; {3, 2} and {3, 4},
// 3000 x 2000 x 200 NT 9.8 and 10.4 us, x 640 13.0 and 13.5, x 1280 19.2 and 19.5, with B out of the caches 22.2 and 21.7).
struct Rings { int a, b; };
constexpr Rings rings(int BM, int BN, bool DEEP) {
  return BM == 256 && BN == 128 && DEEP ? Rings{3, 4} : BM == 192 && BN == 256 ? Rings{2, 3} : (3 * BM + 2 * BN) * BK * 2 <= 160 * 1024 ? Rings{3, 2} : Rings{2, 2};
}
constexpr int ring_bytes(int BM, int BN, bool DEEP) { return (rings(BM, BN, DEEP).a * BM + rings(BM, BN, DEEP).b * BN) * BK * 2; }
inline bool ring_pays(const GemmArgs& a) { return a.K / (a.splits > 1 ? a.splits : 1) >= 2048; }

// KS tile [64 k][R rows]: element (k, n) at byte 2 R k + 64 ((n >> 5) ^ ks_swz(k)) + 2 (n & 31).  A transposing read
// covers 4 consecutive k x 16 n: the XOR, together with the row pitch, puts the 4 rows in 4 different 64-byte quarters of
// the banks.  Two such groups of 16 lanes share a clock of the LDS, and their rows, 8 apart, share quarters: 4.0 clocks a read
// with eight waves reading.  An XOR of 32-byte pieces that parts them too makes it 2.4, but its addresses cost the vector
// ALU more than the LDS gains: products of 256x256 and 256x320 tiles came out level to 2 % slower.
template <int R>
DEV int ks_swz(int k) {
  static_assert(R % 64 == 0, "rows of a contraction-strided tile");
  return R % 128 == 0 ? (k & 3) : ((k >> 1) & 1);
}

// Loads of one operand tile: R rows (columns of C for B), NW waves, IPW one-KiB pieces per wave.
//   KC tile [R rows][64 k]: 16-byte chunk (r, c) at slot 8 r + (c ^ (r & 7)): the 8 lanes that one LDS clock serves in a
//       fragment read (8 rows, one chunk index) touch all banks once, and 8 lanes of a load cover a whole 128-byte line.
//   KS tile [64 k][R rows]: see ks_swz.
// The tile is advanced along the contraction in the buffer resource (base and extent, scalar registers): a load costs
// the vector ALU nothing but the contraction-tail select of a KC operand.
template <int R, int NW, bool KS>
struct TileLoader {
  static_assert(R % (8 * NW) == 0, "tile pieces must divide over the waves");
  static constexpr int IPW = R / 8 / NW;
  uint32_t base[IPW];   // byte offset of the lane's chunk in tile 0, or BUF_OOB
  int kofs;             // KC: contraction offset of the lane's chunk inside the tile
  const char* ptr;      // start of the next tile to be loaded
  int left, step;       // bytes from there to the operand's end; bytes from tile to tile
  int kleft;            // contraction elements from there on

  template <class ColMap>
  DEV void init(const void* p, long bytes, int ld, int K, const ColMap& cols, int row0, int row_end, int wave, int lane) {
    ptr = static_cast<const char*>(p);
    left = (int)bytes;
    step = KS ? BK * ld * 2 : BK * 2;
    kleft = K;
    kofs = ((lane & 7) ^ (lane >> 3)) * 8;
#pragma unroll
    for (int i = 0; i < IPW; ++i) {
      if constexpr (KS) {
        const int P = (wave * IPW + i) * 1024 + lane * 16;
        const int k = P / (R * 2), w = P % (R * 2);
        const int c = cols((((w >> 6) ^ ks_swz<R>(k)) << 5) + ((w >> 4) & 3) * 8);
        base[i] = c >= 0 ? (uint32_t)(k * ld + c) * 2u : BUF_OOB;
      } else {
        const int r = row0 + 8 * (wave * IPW + i) + (lane >> 3);
        base[i] = r < row_end ? (uint32_t)(r * ld + kofs) * 2u : BUF_OOB;
      }
    }
  }
  DEV buf_rsrc rsrc() const { return make_rsrc(ptr, left); }
  DEV bool inside() const { return KS || kofs < kleft; }     // contraction tail: chunks past K load zeros
  DEV void advance(int n = 1) { ptr += (long)n * step; left = left > n * step ? left - n * step : 0; kleft -= n * BK; }
  DEV void issue(int i, buf_rsrc rs, bool in, uint8_t* tile, int wave) const {
    const uint32_t off = KS || in ? base[i] : BUF_OOB;
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, LDS_PTR(tile + (wave * IPW + i) * 1024), 16, off, 0, 0, 0);
  }
};

template <int I, int N, class F>
DEV void static_for(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    static_for<I + 1, N>(f);
  }
}

// Per-lane byte offsets of a 16-row fragment's reads inside a tile: lane holds row lane%16, elements 8 (lane/16) .. of 32.
DEV uint32_t kc_frag_off16(int lane) { const int fr = lane & 15, fh = lane >> 4; return (uint32_t)(fr * 128 + ((fh ^ (fr & 7)) << 4)); }
template <int R>
DEV uint32_t ks_frag_off16(int lane, int n32) {       // of columns 32 n32 .. + 15, first of the two transposing reads; the second is 4 k rows on
  const int fr = lane & 15, fh = lane >> 4, k = 8 * fh + (fr >> 2);
  return (uint32_t)(k * R * 2 + ((n32 ^ ks_swz<R>(k)) << 6) + 8 * (fr & 3));
}

// SwiGLU forward: the tile's even 32-column groups are gate columns, the odd ones the matching
// up columns, so one lane sees gate and up of the same ffn column.
struct GluCols {
  int c0, n_split;
  DEV int operator()(int r) const {
    int col = c0 + ((r >> 6) << 5) + (r & 31);
    if (col >= n_split) return -1;
    return col + ((r >> 5) & 1) * n_split;
  }
};

// Rotary embedding: the partner columns (i, i + d/2) of a head must meet in one lane of the epilogue, which pairs
// tile columns 32 apart inside every 64 (as for SwiGLU).  Heads of 64 columns already lie that way; for
// heads of 128 the second and third group of 32 inside every 128 trade places.
struct RopeCols {
  int n0, n_end, d;
  DEV int at(int r) const {
    const int g = n0 + r;
    return d == 128 ? ((g & ~96) | (((g >> 5) & 1) << 6) | (((g >> 6) & 1) << 5)) : g;
  }
  DEV int operator()(int r) const { const int g = at(r); return g < n_end ? g : -1; }
};

// Epilogue.  Stored from the accumulators, every instruction would touch 16 rows with 32 or 64 bytes each.  Blocks of
// fp32 sums go through LDS instead: written by row owner, read back with WN/4 consecutive lanes along a row, so that
// loads of the side tensors and all stores cover whole 128-byte lines.
constexpr int epi_row_bytes(int WN) { return WN * 4 + 16; }      // padded row: the 16 rows of a write phase hit distinct banks

// what depends on a lane's 4 columns only: lane (row lane / (WN/4) of an instruction) has the 4 from rcol on
template <int BN, int WN, int EPI>
struct EpiCols {
  int rcol, rrow;
  int n, col;                                    // global column; SwiGLU: ffn column of the gate / up pair
  bool n_ok;
  float rfreq[EPI == EPI_ROPE ? 4 : 1];          // rotary embedding: the frequencies of the lane's 4 pair indices
  bool rot;
  f32x4 bias4;

  DEV EpiCols(const GemmArgs& p, int tn, int n0, int wn0, int lane) {
    rrow = lane / (WN / 4);
    rcol = (lane % (WN / 4)) * 4;
    const int nl = wn0 + rcol;                   // tile-local column of the first of this lane's 4
    col = 0; rot = false;
    if constexpr (EPI == EPI_SWIGLU) {
      col = tn * (BN / 2) + ((nl >> 6) << 5) + (nl & 31);
      n = col;
      n_ok = !((nl >> 5) & 1) && col < p.n_split;  // up groups are handled by the lane holding their gate group
    } else if constexpr (EPI == EPI_ROPE) {
      static_assert(EPI != EPI_ROPE || WN % 64 == 0, "the rotary epilogue pairs columns inside 64-column groups");
      n = RopeCols{n0, p.N, p.rope_d}.at(nl);                    // memory column of the first element of the pair
      n_ok = !((nl >> 5) & 1) && n < p.N;                        // the partner groups are handled by the lane holding i
      rot = n_ok && n < p.rope_cols;
#pragma unroll
      for (int e = 0; e < 4; ++e) rfreq[e] = rot ? rope_freq(n % p.rope_d + e, p.rope_d, p.rope_log2_base) : 0.0f;
    } else {
      n = n0 + nl;
      n_ok = n < p.N;
    }
    bias4 = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    if constexpr (EPI == EPI_STORE || EPI == EPI_BIAS_GELU || EPI == EPI_RESID) {
      if (p.bias && n_ok) {
        const u32x2 bb = *reinterpret_cast<const u32x2*>(static_cast<const bf16_t*>(p.bias) + n);
        bias4 = f32x4{bf16_lo(bb[0]), bf16_hi(bb[0]), bf16_lo(bb[1]), bf16_hi(bb[1])};
      }
    }
  }
};

// Stores ROWS rows of sums from LDS.  side() requests what the epilogue needs of the side tensors for the rows from m on
// and is called one block of rows ahead of finish(), which reads the sums and stores: loads of global memory (1 to 2 us)
// are in flight while the block before them is worked on.  Rows or columns outside the matrix read a safe address instead
// of branching, their results are never stored.  The sums of PARTS buffers PART_BYTES apart are added in their order.
template <int BN, int WN, int EPI, int ROWS, int ROW_BYTES = epi_row_bytes(WN), int PARTS = 1, int PART_BYTES = 0>
struct RowStore {
  static constexpr int ROWB = ROW_BYTES, NROWS = ROWS;
  static constexpr int RPI = 64 / (WN / 4);      // rows per read instruction
  static constexpr int NR = ROWS / RPI;          // read-back instructions
  static constexpr bool PAIR = EPI == EPI_SWIGLU || EPI == EPI_ROPE;
  struct Side {
    u32x2 a[(EPI == EPI_DGELU || EPI == EPI_DSWIGLU || EPI == EPI_RESID) ? NR : 1], b[(EPI == EPI_DSWIGLU || EPI == EPI_RESID) ? NR : 1];
    f32x4 old[EPI == EPI_ACC_F32 ? NR : 1];
  };
  const GemmArgs& p;
  const EpiCols<BN, WN, EPI>& ec;

  DEV bool inside(int m, int t, long& row) const {
    const int mr = m + t * RPI + ec.rrow;
    const bool ok = ec.n_ok && mr < p.M;
    row = ok ? (long)mr : 0L;
    return ok;
  }
  DEV void side(Side& s, int m) const {
#pragma unroll
    for (int t = 0; t < NR; ++t) {
      long row;
      const int ns = inside(m, t, row) ? ec.n : 0;
      if constexpr (EPI == EPI_ACC_F32) {
        if (p.beta) s.old[t] = *reinterpret_cast<const f32x4*>(static_cast<const float*>(p.C) + row * p.ldc + ns);
      } else if constexpr (EPI == EPI_DGELU) {
        s.a[t] = *reinterpret_cast<const u32x2*>(static_cast<const bf16_t*>(p.aux) + row * p.ldaux + ns);
      } else if constexpr (EPI == EPI_RESID) {
        s.a[t] = *reinterpret_cast<const u32x2*>(static_cast<const bf16_t*>(p.aux) + row * p.ldaux + ns);
        s.b[t] = u32x2{0u, 0u};
        if (p.add2) s.b[t] = *reinterpret_cast<const u32x2*>(static_cast<const bf16_t*>(p.add2) + row * p.ldaux + ns);
      } else if constexpr (EPI == EPI_DSWIGLU) {
        const bf16_t* aux = static_cast<const bf16_t*>(p.aux) + row * p.ldaux;
        s.a[t] = *reinterpret_cast<const u32x2*>(aux + ns);
        s.b[t] = *reinterpret_cast<const u32x2*>(aux + p.n_split + ns);
      }
    }
  }
  DEV f32x4 read(const uint8_t* buf, int at) const {
    f32x4 part[PARTS];
#pragma unroll
    for (int k = 0; k < PARTS; ++k) part[k] = *reinterpret_cast<const f32x4*>(buf + k * PART_BYTES + at);
    f32x4 v = part[0];
#pragma unroll
    for (int k = 1; k < PARTS; ++k) v += part[k];
    return v;
  }
  // buf: row m's sums
  DEV void finish(const Side& s, const uint8_t* buf, int m) const {
    if constexpr (EPI == EPI_BIAS_GELU || EPI == EPI_DGELU) {
      if (p.gelu_tanh) finish_form<true>(s, buf, m); else finish_form<false>(s, buf, m);
    } else {
      finish_form<true>(s, buf, m);
    }
  }
  template <bool TANH>
  DEV void finish_form(const Side& s, const uint8_t* buf, int m) const {
    const int n = ec.n, col = ec.col;
    f32x4 v[NR], u[PAIR ? NR : 1];
#pragma unroll
    for (int t = 0; t < NR; ++t) {
      const int at = (t * RPI + ec.rrow) * ROWB;
      v[t] = read(buf, at + ec.rcol * 4);
      if constexpr (PAIR) u[t] = read(buf, at + (ec.rcol ^ 32) * 4);
    }
#pragma unroll
    for (int t = 0; t < NR; ++t) {
      long row;
      const bool ok = inside(m, t, row);
      f32x4 w = v[t];
      if constexpr (EPI == EPI_SWIGLU) {
        if (ok) {
          bf16_t* aux = static_cast<bf16_t*>(p.aux) + row * p.ldaux;
          const u32x2 pg = {pack_bf16(w[0], w[1]), pack_bf16(w[2], w[3])};
          const u32x2 pu = {pack_bf16(u[t][0], u[t][1]), pack_bf16(u[t][2], u[t][3])};
          *reinterpret_cast<u32x2*>(aux + col) = pg;
          *reinterpret_cast<u32x2*>(aux + p.n_split + col) = pu;
          f32x4 o;
#pragma unroll
          for (int e = 0; e < 4; ++e) o[e] = w[e] * sigmoid_f(w[e]) * u[t][e];
          const u32x2 po = {pack_bf16(o[0], o[1]), pack_bf16(o[2], o[3])};
          *reinterpret_cast<u32x2*>(static_cast<bf16_t*>(p.C) + row * p.ldc + col) = po;
        }
      } else if constexpr (EPI == EPI_ACC_F32) {
        if (p.beta) w += s.old[t];
        if (ok) *reinterpret_cast<f32x4*>(static_cast<float*>(p.C) + row * p.ldc + n) = w;
      } else if constexpr (EPI == EPI_ROPE) {
        f32x4 hi = u[t];
        if (ec.rot) {
          const float pos = (float)(int)(row % p.rope_seq);
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            float sn, cs;
            rope_sincos(pos, ec.rfreq[e], &sn, &cs);
            const float a = w[e], b = hi[e];
            w[e] = a * cs - b * sn;
            hi[e] = b * cs + a * sn;
          }
        }
        if (ok) {
          bf16_t* crow = static_cast<bf16_t*>(p.C) + row * p.ldc + n;
          const u32x2 plo = {pack_bf16(w[0], w[1]), pack_bf16(w[2], w[3])};
          const u32x2 phi = {pack_bf16(hi[0], hi[1]), pack_bf16(hi[2], hi[3])};
          *reinterpret_cast<u32x2*>(crow) = plo;
          *reinterpret_cast<u32x2*>(crow + (p.rope_d >> 1)) = phi;
        }
      } else if constexpr (EPI == EPI_RESID) {
        // the sum takes the partial sum as it is stored, in the order of the norm kernel that forms it between two blocks
        const u32x2 pp = {pack_bf16(w[0], w[1]), pack_bf16(w[2], w[3])};
        const float x1[4] = {bf16_lo(s.a[t][0]), bf16_hi(s.a[t][0]), bf16_lo(s.a[t][1]), bf16_hi(s.a[t][1])};
        const float part[4] = {bf16_lo(pp[0]), bf16_hi(pp[0]), bf16_lo(pp[1]), bf16_hi(pp[1])};
        const float oth[4] = {bf16_lo(s.b[t][0]), bf16_hi(s.b[t][0]), bf16_lo(s.b[t][1]), bf16_hi(s.b[t][1])};
        float y[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) y[e] = ((x1[e] + part[e]) + oth[e]) + ec.bias4[e];
        const u32x2 py = {pack_bf16(y[0], y[1]), pack_bf16(y[2], y[3])};
        if (ok) {
          *reinterpret_cast<u32x2*>(static_cast<bf16_t*>(p.C) + row * p.ldc + n) = pp;
          *reinterpret_cast<u32x2*>(static_cast<bf16_t*>(p.out2) + row * p.ldaux + n) = py;
        }
      } else {
        w += ec.bias4;
        if constexpr (EPI == EPI_BIAS_GELU) {
          const u32x2 pp = {pack_bf16(w[0], w[1]), pack_bf16(w[2], w[3])};
          if (ok) *reinterpret_cast<u32x2*>(static_cast<bf16_t*>(p.aux) + row * p.ldaux + n) = pp;
#pragma unroll
          for (int e = 0; e < 4; ++e) w[e] = gelu_f<TANH>(w[e]);
        } else if constexpr (EPI == EPI_DGELU) {
          w[0] *= gelu_grad_f<TANH>(bf16_lo(s.a[t][0])); w[1] *= gelu_grad_f<TANH>(bf16_hi(s.a[t][0]));
          w[2] *= gelu_grad_f<TANH>(bf16_lo(s.a[t][1])); w[3] *= gelu_grad_f<TANH>(bf16_hi(s.a[t][1]));
        } else if constexpr (EPI == EPI_DSWIGLU) {
          const float gv[4] = {bf16_lo(s.a[t][0]), bf16_hi(s.a[t][0]), bf16_lo(s.a[t][1]), bf16_hi(s.a[t][1])};
          const float uv[4] = {bf16_lo(s.b[t][0]), bf16_hi(s.b[t][0]), bf16_lo(s.b[t][1]), bf16_hi(s.b[t][1])};
          f32x4 du;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float sg = sigmoid_f(gv[e]);
            du[e] = w[e] * gv[e] * sg;                                   // d_act * silu(g)
            w[e] = w[e] * uv[e] * sg * (1.0f + gv[e] * (1.0f - sg));     // d_act * u * silu'(g)
          }
          const u32x2 pdu = {pack_bf16(du[0], du[1]), pack_bf16(du[2], du[3])};
          if (ok) *reinterpret_cast<u32x2*>(static_cast<bf16_t*>(p.C) + row * p.ldc + p.n_split + n) = pdu;
        }
        const u32x2 po = {pack_bf16(w[0], w[1]), pack_bf16(w[2], w[3])};
        if (ok) *reinterpret_cast<u32x2*>(static_cast<bf16_t*>(p.C) + row * p.ldc + n) = po;
      }
    }
  }
};

// 32 rows of sums in blocks of rows, the side tensors one block ahead; `more`: rows follow.
template <class Store>
DEV void store_rows32(const Store& rs, typename Store::Side& cur, const uint8_t* buf, int m, bool more) {
  typename Store::Side nxt;
#pragma unroll 1
  for (int b = 0; b < 32 / Store::NROWS; ++b) {
    const int mb = m + b * Store::NROWS;
    if (more || b < 32 / Store::NROWS - 1) rs.side(nxt, mb + Store::NROWS);
    rs.finish(cur, buf + b * Store::NROWS * Store::ROWB, mb);
    cur = nxt;
  }
}
constexpr int epi_block_rows(int C) { return 8 * (256 / C) < 32 ? 8 * (256 / C) : 32; }       // eight read instructions, at most 32 rows

// The products of one launch: one, or several weight gradients with tiles first[i] .. first[i + 1] - 1 of the launch each.
// With several contraction ranges (splits) the tiles of range s follow those of range s - 1, it starts s * k_per elements
// down the contraction and its sums go part_stride floats behind the range's before it.
struct GemmGroup { GemmArgs g[GEMM_GROUP]; int first[GEMM_GROUP + 1]; int splits, k_per; long part_stride; };

// The MFMAs of the large tiles are inline assembly, which says where their sums live: 64 accumulators in the 256 accumulation
// registers, what a tile has beyond that in vector registers.  Left to itself the compiler takes the accumulation registers for
// all of them and copies in and out around the loop's ends (24 sums a tile of 256x256) or, beyond 256 registers, around
// every use.  It does not see these instructions' latency: the epilogue keeps its own distance.
constexpr int IN_AGPRS = 64;
DEV void mfma_agpr(bf16x8 a, bf16x8 b, f32x4& c) { asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+a"(c) : "v"(a), "v"(b)); }
DEV void mfma_vgpr(bf16x8 a, bf16x8 b, f32x4& c) { asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(a), "v"(b)); }

template <int BM, int BN, int WM, int WN, bool AKS, bool BKS, int EPI, bool DEEP>
DEV void gemm_body(const GemmArgs& p, const int lin) {
  constexpr int NW = (BM / WM) * (BN / WN);
  constexpr int TM = WM / 16, TN = WN / 16, RING_A = rings(BM, BN, DEEP).a, RING_B = rings(BM, BN, DEEP).b;
  constexpr int A_BYTES = BM * BK * 2, B_BYTES = BN * BK * 2;
  extern __shared__ __align__(1024) uint8_t smem[];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm0 = (wave % (BM / WM)) * WM, wn0 = (wave / (BM / WM)) * WN;

  // bands of group_m tile rows, walked column by column
  const int band = lin / (p.group_m * p.tiles_n), inband = lin % (p.group_m * p.tiles_n);
  const int gm = min(p.group_m, p.tiles_m - band * p.group_m);
  const int tm = band * p.group_m + inband % gm, tn = inband / gm;
  const int m0 = tm * BM, n0 = tn * BN;

  TileLoader<BM, NW, AKS> ldA;
  TileLoader<BN, NW, BKS> ldB;
  constexpr int IPA = TileLoader<BM, NW, AKS>::IPW, IPB = TileLoader<BN, NW, BKS>::IPW;
  ldA.init(p.A, p.a_bytes, (int)p.lda, p.K, IdentityCols{m0, p.M}, m0, p.M, wave, lane);
  if constexpr (EPI == EPI_SWIGLU) ldB.init(p.B, p.b_bytes, (int)p.ldb, p.K, GluCols{tn * (BN / 2), p.n_split}, n0, p.N, wave, lane);
  else if constexpr (EPI == EPI_ROPE) ldB.init(p.B, p.b_bytes, (int)p.ldb, p.K, RopeCols{n0, p.N, p.rope_d}, n0, p.N, wave, lane);
  else ldB.init(p.B, p.b_bytes, (int)p.ldb, p.K, IdentityCols{n0, p.N}, n0, p.N, wave, lane);
  uint8_t* const ringB = smem + RING_A * A_BYTES;

  f32x4 acc[TN][TM];
#pragma unroll
  for (int i = 0; i < TN; ++i)
#pragma unroll
    for (int j = 0; j < TM; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

  // per-lane LDS byte offsets of the fragments inside a tile.  A fragment is 16 rows x 32 contraction elements: lane
  // holds row lane%16, elements 8 (lane/16) ..; the tile's second 32 elements are reached by XOR 64 (KC) or 32 rows on (KS)
  const int fr = lane & 15, fh = lane >> 4;
  const uint32_t kc_off = kc_frag_off16(lane);
  // (KS: groups of 32 columns up to the XOR's period apart have offsets of their own, a multiple of it apart a constant)
  constexpr int GA = BM % 128 == 0 && WM > 64 ? 4 : 2, GB = BN % 128 == 0 && WN > 64 ? 4 : 2;
  uint32_t offA[AKS ? GA : 1], offB[BKS ? GB : 1];
  if constexpr (AKS) {
#pragma unroll
    for (int j = 0; j < GA; ++j) offA[j] = ks_frag_off16<BM>(lane, (wm0 >> 5) + j);
  } else {
    offA[0] = kc_off + wm0 * 128;
  }
  if constexpr (BKS) {
#pragma unroll
    for (int i = 0; i < GB; ++i) offB[i] = ks_frag_off16<BN>(lane, (wn0 >> 5) + i);
  } else {
    offB[0] = kc_off + wn0 * 128;
  }

  // Fragments of the two 32-deep MFMA steps of a tile: those of one step are read while the MFMAs of the other run.  A tile of
  // up to 64 accumulators holds both sets.  The larger ones walk the operand of more fragments in the outer loop of a step
  // and refill a fragment of it in place behind its last MFMA; its last SPARE fragments have a second place each, so that the
  // last reads of a step are some 16 MFMAs ahead of the wait.  The two halves of a transposed fragment stay apart until the
  // wait has passed: joining them earlier could copy a register whose read is still in flight.
  constexpr bool IN_PLACE = TM * TN > 64, OUTER_A = IN_PLACE && TM > TN;
  constexpr int SPARE = 2, NO = OUTER_A ? TM : TN, NI = OUTER_A ? TN : TM;      // fragments of the outer and the inner operand
  constexpr int HA = AKS ? 2 : 1, HB = BKS ? 2 : 1, HO = OUTER_A ? HA : HB, HI = OUTER_A ? HB : HA;      // reads of a fragment
  constexpr int FA = OUTER_A ? TM + SPARE : 2 * TM, FB = IN_PLACE && !OUTER_A ? TN + SPARE : 2 * TN;
  u32x4 fa[AKS ? 1 : FA], fb[BKS ? 1 : FB];
  u32x2 ha[AKS ? FA : 1][2], hb[BKS ? FB : 1][2];
  auto at_a = [](int s, int j) constexpr { return !OUTER_A ? s * TM + j : j < TM - SPARE ? j : j + s * SPARE; };
  auto at_b = [](int s, int i) constexpr { return !IN_PLACE || OUTER_A ? s * TN + i : i < TN - SPARE ? i : i + s * SPARE; };
  auto read_a = [&](auto step, auto frag, auto half, uint32_t ta) {
    constexpr int s = decltype(step)::value, j = decltype(frag)::value, h = decltype(half)::value, at = at_a(s, j);
    if constexpr (AKS) ha[at][h] = ds_read_tr_at<(s * 32 + h * 4) * BM * 2 + (j & 1) * 32 + j / 2 / GA * GA * 64>(ta + offA[j / 2 % GA]);
    else fa[at] = ds_read_b128_at<j * 2048>(ta + (offA[0] ^ (s << 6)));
  };
  auto read_b = [&](auto step, auto frag, auto half, uint32_t tb) {
    constexpr int s = decltype(step)::value, i = decltype(frag)::value, h = decltype(half)::value, at = at_b(s, i);
    if constexpr (BKS) hb[at][h] = ds_read_tr_at<(s * 32 + h * 4) * BN * 2 + (i & 1) * 32 + i / 2 / GB * GB * 64>(tb + offB[i / 2 % GB]);
    else fb[at] = ds_read_b128_at<i * 2048>(tb + (offB[0] ^ (s << 6)));
  };
  auto read_outer = [&](auto step, auto frag, auto half, uint32_t ta, uint32_t tb) {
    if constexpr (OUTER_A) read_a(step, frag, half, ta); else read_b(step, frag, half, tb);
  };
  // reads that no MFMA of the step before holds up: the inner operand, then of the outer one all, or the SPARE in two places
  constexpr int READS = NI * HI + (IN_PLACE ? SPARE : NO) * HO;
  auto read_one = [&](auto step, auto which, uint32_t ta, uint32_t tb) {
    constexpr int r = decltype(which)::value;
    if constexpr (r < NI * HI) {
      using frag = std::integral_constant<int, r / HI>;
      using half = std::integral_constant<int, r % HI>;
      if constexpr (OUTER_A) read_b(step, frag{}, half{}, tb); else read_a(step, frag{}, half{}, ta);
    } else {
      constexpr int q = r - NI * HI;
      read_outer(step, std::integral_constant<int, q / HO + (IN_PLACE ? NO - SPARE : 0)>{}, std::integral_constant<int, q % HO>{}, ta, tb);
    }
  };
  // a wait on the LDS counter followed by "uses and redefinitions" of the fragments: no MFMA can move above it
  auto tie_step = [&](auto step) {
    constexpr int s = decltype(step)::value;
    lds_wait<0>();
#pragma unroll
    for (int j = 0; j < TM; ++j) {
      if constexpr (AKS) { tie(ha[at_a(s, j)][0]); tie(ha[at_a(s, j)][1]); } else tie(fa[at_a(s, j)]);
    }
#pragma unroll
    for (int i = 0; i < TN; ++i) {
      if constexpr (BKS) { tie(hb[at_b(s, i)][0]); tie(hb[at_b(s, i)][1]); } else tie(fb[at_b(s, i)]);
    }
  };
  auto frag_a = [&](int s, int j) {
    const int k = at_a(s, j);
    if constexpr (AKS) return __builtin_bit_cast(bf16x8, u32x4{ha[k][0][0], ha[k][0][1], ha[k][1][0], ha[k][1][1]});
    else return __builtin_bit_cast(bf16x8, fa[k]);
  };
  auto frag_b = [&](int s, int i) {
    const int k = at_b(s, i);
    if constexpr (BKS) return __builtin_bit_cast(bf16x8, u32x4{hb[k][0][0], hb[k][0][1], hb[k][1][0], hb[k][1][1]});
    else return __builtin_bit_cast(bf16x8, fb[k]);
  };
  // MFMA m of step s, and the reads for the other step that follow it
  auto mfma_and_reads = [&](auto step, auto next, auto mc, uint32_t ta, uint32_t tb) {
    constexpr int s = decltype(step)::value, m = decltype(mc)::value, o = m / NI, i = OUTER_A ? m % NI : o, j = OUTER_A ? o : m % NI;
    constexpr int EVERY = TM * TN * 3 / 4 / READS > 0 ? TM * TN * 3 / 4 / READS : 1;      // MFMAs per LDS read
    if constexpr (m >= IN_AGPRS) mfma_vgpr(frag_b(s, i), frag_a(s, j), acc[i][j]);
    else if constexpr (TM * TN > 16) mfma_agpr(frag_b(s, i), frag_a(s, j), acc[i][j]);
    else acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(frag_b(s, i), frag_a(s, j), acc[i][j], 0, 0, 0);
    if constexpr (m % EVERY == 0 && m / EVERY < READS) read_one(next, std::integral_constant<int, m / EVERY>{}, ta, tb);
    if constexpr (IN_PLACE && o > 0 && o <= NO - SPARE && (m % NI == 1 || (HO == 2 && m % NI == 3)))
      read_outer(next, std::integral_constant<int, o - 1>{}, std::integral_constant<int, m % NI / 2>{}, ta, tb);
  };
  using step0 = std::integral_constant<int, 0>;
  using step1 = std::integral_constant<int, 1>;

  // X: the operand with more places, loaded during step 0 into the place of the tile before; Y: the other one, during step 1
  constexpr bool X_IS_B = RING_B > RING_A, BOTH = RING_A == RING_B;

  // Software pipeline.  Tile kt's two MFMA steps: during step 0 the fragments of step 1 are read, during step 1 those
  // of tile kt+1's step 0.  The one barrier of a tile stands between the steps: by then every wave has read all of tile
  // kt, whose two ring places are refilled from there on: Y's during step 1 with tile kt+Y, X's during the next tile's
  // step 0 with tile kt+X (X and Y for the number of places of each).  So loads are spread over the whole tile, in 256x256 one
  // every 8 MFMAs (a load occupies the address path for 16 clocks; bunched up behind the barrier they stall the MFMAs issued
  // between them), and with three and two places each has at least a step to land, with four and three three.  Where the LDS
  // has two places of each only (tiles of 320), both are loaded during step 1, A first, which comes from further away: one every
  // 3 MFMAs (every 2 measured 3 to 4 % slower); a step of such a tile is a quarter longer, which is what its loads have less to land in.
  // (8192^3, N(0,1) x N(0,0.02), NT / NN / TN: 1.52 / 1.53 / 1.48 PFLOP/s; with compiler-placed sums 1.51 / 1.49 / 1.43, and on
  // another board 1.48 / 1.45 / 1.43, where a ring of four 32-deep tiles, eight waves and 32x32x16 MFMAs made 1.20 / 1.26 /
  // 1.21 and two rings of two 1.42 / 1.39 / 1.40.)
  const int nk = (p.K + BK - 1) / BK;
  auto fill_a = [&](int slot) {
    const buf_rsrc rs = ldA.rsrc();
    const bool in = ldA.inside();
#pragma unroll
    for (int i = 0; i < IPA; ++i) ldA.issue(i, rs, in, smem + slot * A_BYTES, wave);
    ldA.advance();
  };
  auto fill_b = [&](int slot) {
    const buf_rsrc rs = ldB.rsrc();
    const bool in = ldB.inside();
#pragma unroll
    for (int i = 0; i < IPB; ++i) ldB.issue(i, rs, in, ringB + slot * B_BYTES, wave);
    ldB.advance();
  };
  // The loads in the order that the loop goes on with, the first tile's in front.  BEHIND: loads asked for behind those of tile
  // kt+1 when the barrier of tile kt is reached; X(kt+1) was asked for 2 (X - 2) steps before that one, Y(kt+1) 2 Y - 3.
  constexpr int X = X_IS_B ? RING_B : RING_A, Y = X_IS_B ? RING_A : RING_B, IPX = X_IS_B ? IPB : IPA, IPY = X_IS_B ? IPA : IPB;
  auto fill_x = [&](int slot) { if constexpr (X_IS_B) fill_b(slot); else fill_a(slot); };
  auto fill_y = [&](int slot) { if constexpr (X_IS_B) fill_a(slot); else fill_b(slot); };
  constexpr int SINCE = 2 * Y - 3 < 2 * (X - 2) ? 2 * Y - 3 : 2 * (X - 2);
  constexpr int BEHIND = BOTH ? 0 : (SINCE + 1) / 2 * IPX + SINCE / 2 * IPY;
  if constexpr (BOTH) {
    fill_x(0); fill_y(0); fill_x(1); fill_y(1);
    wait_vmcnt<IPX + IPY>();
  } else {
    static_assert(X == Y + 1, "the order of the loads in front of the loop");
    static_for<0, Y>([&](auto t) { fill_x(decltype(t)::value); fill_y(decltype(t)::value); });
    wait_vmcnt<(Y - 1) * (IPX + IPY)>();
  }
  __builtin_amdgcn_s_barrier();
  const uint32_t lds_a = lds_addr(smem), lds_b = lds_addr(ringB);
  static_for<0, READS>([&](auto r) { read_one(step0{}, r, lds_a, lds_b); });
  if constexpr (IN_PLACE) {
    static_for<0, (NO - SPARE) * HO>([&](auto r) {
      read_outer(step0{}, std::integral_constant<int, decltype(r)::value / HO>{}, std::integral_constant<int, decltype(r)::value % HO>{}, lds_a, lds_b);
    });
  }

  constexpr int NM = TM * TN;                          // MFMAs per step
  int sa = 0, sb = 0;                                  // ring places of tile kt
  int free_x = X - 1;                                  // ring place that tile kt-1 left to the tile of X loaded in step 0
  for (int kt = 0; kt < nk; ++kt) {
    const uint32_t ta = lds_a + sa * A_BYTES, tb = lds_b + sb * B_BYTES;
    const int sa_next = sa == RING_A - 1 ? 0 : sa + 1, sb_next = sb == RING_B - 1 ? 0 : sb + 1;
    const uint32_t ta_next = lds_a + sa_next * A_BYTES, tb_next = lds_b + sb_next * B_BYTES;
    tie_step(step0{});
    __builtin_amdgcn_sched_barrier(0);
    {
      const buf_rsrc rs = X_IS_B ? ldB.rsrc() : ldA.rsrc();
      const bool in = X_IS_B ? ldB.inside() : ldA.inside();
      uint8_t* dst = X_IS_B ? ringB + free_x * B_BYTES : smem + free_x * A_BYTES;
      static_for<0, NM>([&](auto mc) {
        constexpr int m = decltype(mc)::value;
        mfma_and_reads(step0{}, step1{}, mc, ta, tb);
        constexpr int LE = NM / IPX;
        if constexpr (!BOTH && m % LE == LE / 2 && m / LE < IPX) {
          if constexpr (X_IS_B) ldB.issue(m / LE, rs, in, dst, wave); else ldA.issue(m / LE, rs, in, dst, wave);
        }
        __builtin_amdgcn_sched_barrier(0);
      });
      if constexpr (!BOTH) { if constexpr (X_IS_B) ldB.advance(); else ldA.advance(); }
    }
    wait_vmcnt<BEHIND>();                              // tile kt+1 has landed (this wave's share); later ones may be in flight
    tie_step(step1{});                                 // ... and this wave has read all of tile kt
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    {
      const buf_rsrc rsb = ldB.rsrc(), rsa = ldA.rsrc();
      const bool inb = ldB.inside(), ina = ldA.inside();
      uint8_t *dstb = ringB + sb * B_BYTES, *dsta = smem + sa * A_BYTES;
      static_for<0, NM>([&](auto mc) {
        constexpr int m = decltype(mc)::value;
        mfma_and_reads(step1{}, step0{}, mc, ta_next, tb_next);
        constexpr int LOADS = BOTH ? IPA + IPB : IPY, LE = BOTH ? NM * 3 / 4 / LOADS : NM / LOADS;
        if constexpr (m % LE == LE / 2 && m / LE < LOADS) {
          constexpr int l = m / LE, a = BOTH || X_IS_B ? IPA : 0;
          if constexpr (l < a) ldA.issue(l, rsa, ina, dsta, wave);
          else ldB.issue(l - a, rsb, inb, dstb, wave);
        }
        __builtin_amdgcn_sched_barrier(0);
      });
      if constexpr (BOTH || !X_IS_B) ldB.advance();
      if constexpr (BOTH || X_IS_B) ldA.advance();
    }
    free_x = X_IS_B ? sb : sa;
    sa = sa_next; sb = sb_next;
  }
  wait_vmcnt<0>();     // the zero-fill loads issued past the last tile must land before the LDS is released
  // The last iteration's look-ahead reads are still in flight: they must land in their registers
  // before the epilogue may reuse those registers.
  tie_step(step0{});
  __builtin_amdgcn_sched_barrier(0);
  if constexpr (TM * TN > 16) asm volatile("s_nop 7\n\ts_nop 7");      // the last sums are 8 wait states away from their MFMA
  __builtin_amdgcn_sched_barrier(0);

  // ---- epilogue.  Accumulator (i, j) value v of a lane is C[m][n] with
  //      m = m0 + wm0 + 16 j + lane%16,  n = n0 + wn0 + 16 i + 4 (lane/16) + v:
  // each wave turns its 32 x WN blocks through its own piece of the (now free) LDS
  __builtin_amdgcn_s_barrier();                  // every wave has finished reading the operand stages
  constexpr int ROWB = epi_row_bytes(WN);
  uint8_t* wbuf = smem + wave * (32 * ROWB);
  // columns in parts whose lanes divide a wave: 128 or 64, and 32 behind them where the wave tile is 160 or 96 wide
  constexpr int CA = WN >= 128 ? 128 : 64, CB = WN - CA;
  const EpiCols<BN, CA, EPI> ec_a(p, tn, n0, wn0, lane);
  const EpiCols<BN, CB ? CB : CA, EPI> ec_b(p, tn, n0, wn0 + (CB ? CA : 0), lane);
  using StoreA = RowStore<BN, CA, EPI, epi_block_rows(CA), ROWB>;
  using StoreB = RowStore<BN, CB ? CB : CA, EPI, epi_block_rows(CB ? CB : CA), ROWB>;
  const StoreA rs_a{p, ec_a};
  const StoreB rs_b{p, ec_b};
  typename StoreA::Side side_a;
  typename StoreB::Side side_b;
  rs_a.side(side_a, m0 + wm0);
  if constexpr (CB > 0) rs_b.side(side_b, m0 + wm0);
  static_for<0, TM / 2>([&](auto jc) __attribute__((always_inline)) {
    constexpr int j = decltype(jc)::value;
#pragma unroll
    for (int i = 0; i < TN; ++i)
#pragma unroll
      for (int g = 0; g < 2; ++g)
        *reinterpret_cast<f32x4*>(wbuf + (16 * g + fr) * ROWB + (i * 16 + fh * 4) * 4) = acc[i][2 * j + g];
    store_rows32(rs_a, side_a, wbuf, m0 + wm0 + j * 32, j < TM / 2 - 1);
    if constexpr (CB > 0) store_rows32(rs_b, side_b, wbuf + CA * 4, m0 + wm0 + j * 32, j < TM / 2 - 1);
  });
}

// Products of few tiles: one workgroup per tile of R x R, the contraction dealt over its waves (wave w of W takes the
// 64-deep operand tiles w, w + W, ...), their sums added in wave order through LDS.  Such launches are bound by the serial
// chain along the contraction, not by any unit's rate: W chains run side by side here, each wave stages its own operand
// tiles (no barrier in the loop), and a tile's loads are in flight while the wave's MFMAs on the one before run.  A wave's
// fragments of both steps sit in registers, so its one stage is free as soon as they are read.
//   64x64, eight waves: for the fewest tiles
//   128x128, four waves: reads half the LDS bytes per MFMA of four waves of 64x64 each
template <int R> struct Split {
  static constexpr int W = R == 64 ? 8 : 4;
  static constexpr int ROWS = 64;                                   // rows of sums that meet in LDS at once
  static constexpr int TILE = R * BK * 2, SUMS = ROWS * epi_row_bytes(R);
  static constexpr int STAGE = SUMS > 2 * TILE ? SUMS : 2 * TILE;   // a wave's LDS: two operand tiles, sums afterwards
  static_assert(STAGE % 1024 == 0 && W * STAGE <= 160 * 1024, "LDS");
};
template <int R, bool AKS, bool BKS, int EPI>
DEV void gemm_split_body(const GemmArgs& p, const int lin) {
  using S = Split<R>;
  constexpr int T = R / 16, NL = R / 8;                             // fragments of a tile; loads of an operand tile
  extern __shared__ __align__(1024) uint8_t smem[];
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int band = lin / (p.group_m * p.tiles_n), inband = lin % (p.group_m * p.tiles_n);
  const int gm = min(p.group_m, p.tiles_m - band * p.group_m);
  const int tm = band * p.group_m + inband % gm, tn = inband / gm;
  const int m0 = tm * R, n0 = tn * R;

  TileLoader<R, 1, AKS> ldA;
  TileLoader<R, 1, BKS> ldB;
  ldA.init(p.A, p.a_bytes, (int)p.lda, p.K, IdentityCols{m0, p.M}, m0, p.M, 0, lane);
  if constexpr (EPI == EPI_SWIGLU) ldB.init(p.B, p.b_bytes, (int)p.ldb, p.K, GluCols{tn * (R / 2), p.n_split}, n0, p.N, 0, lane);
  else if constexpr (EPI == EPI_ROPE) ldB.init(p.B, p.b_bytes, (int)p.ldb, p.K, RopeCols{n0, p.N, p.rope_d}, n0, p.N, 0, lane);
  else ldB.init(p.B, p.b_bytes, (int)p.ldb, p.K, IdentityCols{n0, p.N}, n0, p.N, 0, lane);
  ldA.advance(wave);
  ldB.advance(wave);
  uint8_t* const stage = smem + wave * S::STAGE;
  auto fill = [&] {
    const buf_rsrc ra = ldA.rsrc(), rb = ldB.rsrc();
    const bool ia = ldA.inside(), ib = ldB.inside();
#pragma unroll
    for (int i = 0; i < NL; ++i) ldA.issue(i, ra, ia, stage, 0);
#pragma unroll
    for (int i = 0; i < NL; ++i) ldB.issue(i, rb, ib, stage + S::TILE, 0);
    ldA.advance(S::W);
    ldB.advance(S::W);
  };

  f32x4 acc[T][T];
#pragma unroll
  for (int i = 0; i < T; ++i)
#pragma unroll
    for (int j = 0; j < T; ++j) acc[i][j] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  uint32_t offA[AKS ? T / 2 : 1], offB[BKS ? T / 2 : 1];
  const uint32_t lds_a = lds_addr(stage), lds_b = lds_a + S::TILE;
#pragma unroll
  for (int j = 0; j < (AKS ? T / 2 : 1); ++j) offA[j] = lds_a + (AKS ? ks_frag_off16<R>(lane, j) : kc_frag_off16(lane));
#pragma unroll
  for (int i = 0; i < (BKS ? T / 2 : 1); ++i) offB[i] = lds_b + (BKS ? ks_frag_off16<R>(lane, i) : kc_frag_off16(lane));

  constexpr int ROWB = epi_row_bytes(R), MINE = S::ROWS / S::W;
  const int nk = (p.K + BK - 1) / BK;
  if (wave < nk) fill();
  // what the epilogue reads besides the sums is asked for here where the registers hold it: it is then there with the first tiles
  constexpr bool EARLY = R == 64;
  const EpiCols<R, R, EPI> ec(p, tn, n0, 0, lane);
  using Store = RowStore<R, R, EPI, MINE, ROWB, S::W, S::STAGE>;
  const Store rs{p, ec};
  typename Store::Side side;
  if constexpr (EARLY) rs.side(side, m0 + wave * MINE);
  for (int kt = wave; kt < nk; kt += S::W) {
    u32x4 fa[2][AKS ? 1 : T], fb[2][BKS ? 1 : T];
    u32x2 ha[2][AKS ? T : 1][2], hb[2][BKS ? T : 1][2];
    wait_vmcnt<0>();
    static_for<0, 2>([&](auto sc) {
      constexpr int s = decltype(sc)::value;
      static_for<0, T>([&](auto rc) {
        constexpr int r = decltype(rc)::value;
        if constexpr (AKS) {
          ha[s][r][0] = ds_read_tr_at<s * 32 * R * 2 + (r & 1) * 32>(offA[r / 2]);
          ha[s][r][1] = ds_read_tr_at<(s * 32 + 4) * R * 2 + (r & 1) * 32>(offA[r / 2]);
        } else {
          fa[s][r] = ds_read_b128_at<r * 2048>(lds_a + ((offA[0] - lds_a) ^ (s << 6)));
        }
        if constexpr (BKS) {
          hb[s][r][0] = ds_read_tr_at<s * 32 * R * 2 + (r & 1) * 32>(offB[r / 2]);
          hb[s][r][1] = ds_read_tr_at<(s * 32 + 4) * R * 2 + (r & 1) * 32>(offB[r / 2]);
        } else {
          fb[s][r] = ds_read_b128_at<r * 2048>(lds_b + ((offB[0] - lds_b) ^ (s << 6)));
        }
      });
    });
    lds_wait<0>();
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int r = 0; r < T; ++r) {
        if constexpr (AKS) { tie(ha[s][r][0]); tie(ha[s][r][1]); } else tie(fa[s][r]);
        if constexpr (BKS) { tie(hb[s][r][0]); tie(hb[s][r][1]); } else tie(fb[s][r]);
      }
    if (kt + S::W < nk) fill();
#pragma unroll
    for (int s = 0; s < 2; ++s)
#pragma unroll
      for (int i = 0; i < T; ++i)
#pragma unroll
        for (int j = 0; j < T; ++j) {
          u32x4 a, b;
          if constexpr (AKS) a = u32x4{ha[s][j][0][0], ha[s][j][0][1], ha[s][j][1][0], ha[s][j][1][1]}; else a = fa[s][j];
          if constexpr (BKS) b = u32x4{hb[s][i][0][0], hb[s][i][0][1], hb[s][i][1][0], hb[s][i][1][1]}; else b = fb[s][i];
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, b), __builtin_bit_cast(bf16x8, a), acc[i][j], 0, 0, 0);
        }
  }
  // the sums replace the wave's own operand tiles, 64 rows at a time; then every wave stores its share of these rows.  A wave
  // without a tile (a short contraction) puts down its zeros, so that all the sums of a row are asked for at once
  static_for<0, R / S::ROWS>([&](auto bc) {
    constexpr int B = decltype(bc)::value;
    const int m = m0 + B * S::ROWS + wave * MINE;
    if constexpr (!EARLY) rs.side(side, m);
    if constexpr (B > 0) __syncthreads();                           // everybody has read the rows before
#pragma unroll
    for (int i = 0; i < T; ++i)
#pragma unroll
      for (int j = 0; j < S::ROWS / 16; ++j)
        *reinterpret_cast<f32x4*>(stage + (16 * j + (lane & 15)) * ROWB + (i * 16 + (lane >> 4) * 4) * 4) = acc[i][B * (S::ROWS / 16) + j];
    __syncthreads();
    rs.finish(side, smem + wave * MINE * ROWB, m);
  });
}

// Workgroup ids go round-robin over the 8 XCDs (each with its own L2): every XCD gets one contiguous chunk of the tile
// order, so that the tiles sharing an L2 share operand panels.  Launches of a few tiles keep the plain order, which
// spreads them over all XCDs.
DEV int tile_of_block(int T) {
  if (T < 16) return blockIdx.x;
  return (blockIdx.x & 7) * ((T + 7) >> 3) + (blockIdx.x >> 3);
}

// wave tile = tile: the contraction is dealt over the waves (gemm_split_body)
constexpr int gemm_threads(int BM, int BN, int WM, int WN) { return BM == WM && BN == WN ? (BM == 64 ? Split<64>::W : Split<128>::W) * 64 : (BM / WM) * (BN / WN) * 64; }

template <int BM, int BN, int WM, int WN, bool AKS, bool BKS, int EPI, bool DEEP>
__global__ __launch_bounds__(gemm_threads(BM, BN, WM, WN), BM * BN == 128 * 128 && BM != WM ? 2 : 1)
void gemm_kernel(const GemmArgs p) {
  const int T = p.tiles_m * p.tiles_n, lin = tile_of_block(T);
  if (lin >= T) return;
  if constexpr (BM == WM && BN == WN) gemm_split_body<BM, AKS, BKS, EPI>(p, lin);
  else gemm_body<BM, BN, WM, WN, AKS, BKS, EPI, DEEP>(p, lin);
}

// Several weight gradients of one block in one launch: alone, each leaves part of the chip idle (the 13B shard's are 200,
// 200, 60 and 160 tiles of 256x256 on 256 compute units), and a small block pays mostly for the launches.
template <int BM, int BN, int WM, int WN, bool AKS, bool BKS, int EPI, bool DEEP>
DEV void gemm_group_body(const GemmGroup& p) {
  const int T1 = p.first[GEMM_GROUP], T = T1 * p.splits;
  int lin = tile_of_block(T);
  if (lin >= T) return;
  const int range = lin / T1;
  lin -= range * T1;
  int i = 0;
#pragma unroll
  for (int k = 1; k < GEMM_GROUP; ++k)
    if (lin >= p.first[k]) i = k;
  GemmArgs a = p.g[i];
  const long k0 = (long)range * p.k_per;
  a.A = static_cast<const bf16_t*>(a.A) + k0 * a.lda;
  a.B = static_cast<const bf16_t*>(a.B) + k0 * a.ldb;
  a.a_bytes -= k0 * a.lda * 2;
  a.b_bytes -= k0 * a.ldb * 2;
  a.K = min(a.K - (int)k0, p.k_per);
  a.C = static_cast<float*>(a.C) + range * p.part_stride;
  if constexpr (BM == WM && BN == WN) gemm_split_body<BM, AKS, BKS, EPI>(a, lin - p.first[i]);
  else gemm_body<BM, BN, WM, WN, AKS, BKS, EPI, DEEP>(a, lin - p.first[i]);
}
template <int BM, int BN, int WM, int WN, bool AKS, bool BKS, int EPI, bool DEEP>
__global__ __launch_bounds__(gemm_threads(BM, BN, WM, WN), BM * BN == 128 * 128 && BM != WM ? 2 : 1)
void gemm_group_kernel(const GemmGroup p) {
  gemm_group_body<BM, BN, WM, WN, AKS, BKS, EPI, DEEP>(p);
}

// ... and with further workgroups behind the tiles: in a small block those of the Norm1 backward, then in any block those of
// the bias gradients (four waves each, two to a workgroup of eight).  A dependent launch costs such a block some 4 us whatever it does, and
// its products leave part of the chip idle (forward + backward, us, apart and joined: 256 tokens of a 256-wide block 82 and 73, 1024
// of a 1024-wide one 128 and 117, 4096 of it 241 and 230, 8192 403 and 394, 400 of a Llama one 129 and 125; 256 of a 2048-wide one
// 128 and 120, 2000 of it 228 and 216, 4000 355 and 348; the bias gradients alone: 6018 tokens of the 2.7B shard, whose 224 tiles leave 32
// compute units to them, 626 and 613, 16384 of it 1432 and 1420, 2048 of 13B 650 and 647).
struct GemmTail { HeldTail t; int tiles, norm_blocks, sum_items[COLSUM_MAX_HELD]; };      // workgroups of the tiles and of the norm; column blocks x ranges
template <int BM, int BN, int WM, int WN, bool AKS, bool BKS, int EPI, bool DEEP>
__global__ __launch_bounds__(gemm_threads(BM, BN, WM, WN), BM * BN == 128 * 128 && BM != WM ? 2 : 1)
void gemm_tail_kernel(const GemmGroup p, const GemmTail tail) {
  extern __shared__ __align__(1024) uint8_t smem[];
  if ((int)blockIdx.x < tail.tiles) {
    gemm_group_body<BM, BN, WM, WN, AKS, BKS, EPI, DEEP>(p);
    return;
  }
  const int at = blockIdx.x - tail.tiles;
  float* const lds = reinterpret_cast<float*>(smem);
  if (at < tail.norm_blocks) {
    if (tail.t.norm.rms) norm_bwd_body<2, true, false, false>(tail.t.norm, at, tail.norm_blocks, lds);
    else norm_bwd_body<2, false, false, false>(tail.t.norm, at, tail.norm_blocks, lds);
    return;
  }
  const int wave = threadIdx.x >> 6, quad = wave >> 2;
  int item = (at - tail.norm_blocks) * (gemm_threads(BM, BN, WM, WN) / 256) + quad, k = 0;
  if (item >= tail.sum_items[0]) { item -= tail.sum_items[0]; k = 1; }
  const bool any = item < tail.sum_items[k];
  const ColsumPartial c = tail.t.sums[k];
  colsum_partial_body(static_cast<const bf16_t*>(c.g), c.ld, any ? c.rows : 0, any ? c.n : 0, c.part, item / COLSUM_PARTS, item % COLSUM_PARTS,
                      COLSUM_PARTS, wave & 3, lds + quad * (COLSUM_LDS / 4));
}

// The ranges' sums added in order (and to what the gradient held): HBM-bound, one 16-byte chunk of every range per thread.
struct SplitSum { float* out[GEMM_GROUP]; long end[GEMM_GROUP]; const float* part; long part_stride; int splits, beta; };
__global__ __launch_bounds__(256)
void split_sum_kernel(const SplitSum p) {
  const long at = ((long)blockIdx.x * 256 + threadIdx.x) * 4;
  if (at >= p.part_stride) return;
  float* out = p.out[0] + at;
#pragma unroll
  for (int k = 1; k < GEMM_GROUP; ++k)
    if (at >= p.end[k - 1]) out = p.out[k] + (at - p.end[k - 1]);
  f32x4 v[GEMM_MAX_SPLITS];
#pragma unroll
  for (int s = 0; s < GEMM_MAX_SPLITS; ++s)
    if (s < p.splits) v[s] = *reinterpret_cast<const f32x4*>(p.part + s * p.part_stride + at);
  f32x4 sum = v[0];
#pragma unroll
  for (int s = 1; s < GEMM_MAX_SPLITS; ++s)
    if (s < p.splits) sum += v[s];
  if (p.beta) sum += *reinterpret_cast<const f32x4*>(out);
  *reinterpret_cast<f32x4*>(out) = sum;
}

// fills what the kernel needs to know about the tiles; false: an operand reaches 2 GiB
template <int BM, int BN, bool AKS, bool BKS, int EPI>
bool plan_tiles(GemmArgs& a) {
  const int n_logical = (EPI == EPI_SWIGLU) ? 2 * a.n_split : a.N;
  a.a_bytes = AKS ? ((long)(a.K - 1) * a.lda + a.M) * 2 : ((long)(a.M - 1) * a.lda + a.K) * 2;
  a.b_bytes = BKS ? ((long)(a.K - 1) * a.ldb + n_logical) * 2 : ((long)(a.N - 1) * a.ldb + a.K) * 2;
  a.tiles_m = (a.M + BM - 1) / BM;
  a.tiles_n = (n_logical + BN - 1) / BN;
  a.group_m = a.tiles_m * a.tiles_n >= 16 ? 4 : a.tiles_m;
  return a.a_bytes < (1L << 31) && a.b_bytes < (1L << 31);
}

template <int BM, int BN, int WM, int WN, bool AKS, bool BKS, int EPI, bool DEEP>
hipError_t launch_cfg(const GemmArgs* products, int n, hipStream_t stream) {
  constexpr int NT = gemm_threads(BM, BN, WM, WN);
  constexpr int LDS = BM == WM && BN == WN ? Split<BM == 64 ? 64 : 128>::W * Split<BM == 64 ? 64 : 128>::STAGE : ring_bytes(BM, BN, DEEP);
  auto grid = [](int T) { return dim3(T < 16 ? T : 8 * ((T + 7) / 8)); };
  if (n > 1 || products[0].splits > 1 || products[0].tail) {
    if constexpr (EPI == EPI_ACC_F32 && !(BM == 128 && BN == 256)) {      // (the rule, which alone forms groups, never picks 128x256)
      auto kern = gemm_group_kernel<BM, BN, WM, WN, AKS, BKS, EPI, DEEP>;
      static LdsLimitOnce lds_limit;      // one per instantiation
      if (hipError_t e = lds_limit.ensure(reinterpret_cast<const void*>(kern), LDS); e != hipSuccess) return e;
      GemmGroup grp{};
      SplitSum sum{};
      grp.splits = products[0].splits > 1 ? products[0].splits : 1;
      grp.k_per = ((products[0].K + BK - 1) / BK + grp.splits - 1) / grp.splits * BK;
      grp.splits = (products[0].K + grp.k_per - 1) / grp.k_per;      // no range is empty
      sum.part = products[0].split_ws; sum.splits = grp.splits; sum.beta = products[0].beta;
      int T = 0;
      long at = 0;
      for (int i = 0; i < GEMM_GROUP; ++i) {
        grp.first[i] = T;
        sum.end[i] = at;
        if (i >= n) continue;
        GemmArgs& g = grp.g[i];
        g = products[i];
        if (!plan_tiles<BM, BN, AKS, BKS, EPI>(g) || g.K != products[0].K) return hipErrorInvalidValue;
        T += g.tiles_m * g.tiles_n;
        if (grp.splits > 1) {
          if (g.ldc != g.N || g.beta != sum.beta || !g.split_ws) return hipErrorInvalidValue;
          sum.out[i] = static_cast<float*>(g.C);
          g.C = g.split_ws + at;
          g.beta = 0;
          at += (long)g.M * g.N;
          sum.end[i] = at;
        }
      }
      for (int i = n; i <= GEMM_GROUP; ++i) grp.first[i] = T;
      grp.part_stride = sum.part_stride = at;
      if (products[0].tail) {
        GemmTail tail{};
        tail.t = t_tail;
        t_tail.open = false;
        tail.tiles = (int)grid(T * grp.splits).x;
        tail.norm_blocks = tail.t.norm.rows ? tail.t.norm.slice_blocks * (tail.t.norm.rows / tail.t.norm.slice_rows) : 0;
        for (int k = 0; k < tail.t.nsums; ++k) tail.sum_items[k] = (tail.t.sums[k].n / 8 + 63) / 64 * COLSUM_PARTS;
        constexpr int QUADS = NT / 256;
        const int sums = (tail.sum_items[0] + tail.sum_items[1] + QUADS - 1) / QUADS;
        auto both = gemm_tail_kernel<BM, BN, WM, WN, AKS, BKS, EPI, DEEP>;
        static LdsLimitOnce tail_limit;
        if (hipError_t e = tail_limit.ensure(reinterpret_cast<const void*>(both), LDS); e != hipSuccess) return e;
        hipLaunchKernelGGL(both, dim3(tail.tiles + tail.norm_blocks + sums), dim3(NT), LDS, stream, grp, tail);
      } else {
        hipLaunchKernelGGL(kern, grid(T * grp.splits), dim3(NT), LDS, stream, grp);
      }
      if (hipError_t e = hipGetLastError(); e != hipSuccess || grp.splits == 1) return e;
      hipLaunchKernelGGL(split_sum_kernel, dim3((unsigned)((at / 4 + 255) / 256)), dim3(256), 0, stream, sum);
      return hipGetLastError();
    }
    return hipErrorInvalidValue;
  }
  GemmArgs a = products[0];
  if (!plan_tiles<BM, BN, AKS, BKS, EPI>(a)) return hipErrorInvalidValue;
  auto kern = gemm_kernel<BM, BN, WM, WN, AKS, BKS, EPI, DEEP>;
  static LdsLimitOnce lds_limit;      // one per instantiation
  if (hipError_t e = lds_limit.ensure(reinterpret_cast<const void*>(kern), LDS); e != hipSuccess) return e;
  hipLaunchKernelGGL(kern, grid(a.tiles_m * a.tiles_n), dim3(NT), LDS, stream, a);
  return hipGetLastError();
}

template <bool AKS, bool BKS, int EPI>
hipError_t launch_layout(const GemmArgs* a, int n, int tile_cfg, hipStream_t stream) {
  constexpr bool PAIRED = EPI == EPI_SWIGLU || EPI == EPI_ROPE;      // column pairs 32 apart inside every 64 of a wave tile
  switch (tile_cfg) {
    case GEMM_TILE_256x256: return launch_cfg<256, 256, 128, 128, AKS, BKS, EPI, false>(a, n, stream);
    case GEMM_TILE_256x128:
      if (ring_pays(a[0])) return launch_cfg<256, 128, 128, 64, AKS, BKS, EPI, true>(a, n, stream);
      return launch_cfg<256, 128, 128, 64, AKS, BKS, EPI, false>(a, n, stream);
    // by number only, through the single-kernel entry points, which offer no block output
    case GEMM_TILE_128x256: if constexpr (EPI != EPI_RESID) return launch_cfg<128, 256, 64, 128, AKS, BKS, EPI, false>(a, n, stream); return hipErrorInvalidValue;
    case GEMM_TILE_256x192: if constexpr (!PAIRED) return launch_cfg<256, 192, 128, 96, AKS, BKS, EPI, false>(a, n, stream); return hipErrorInvalidValue;
    case GEMM_TILE_256x320: if constexpr (!PAIRED && EPI != EPI_RESID) return launch_cfg<256, 320, 128, 160, AKS, BKS, EPI, false>(a, n, stream); return hipErrorInvalidValue;
    case GEMM_TILE_192x256: return launch_cfg<192, 256, 96, 128, AKS, BKS, EPI, false>(a, n, stream);
    case GEMM_TILE_320x256: return launch_cfg<320, 256, 160, 128, AKS, BKS, EPI, false>(a, n, stream);
    case GEMM_TILE_64x64:   return launch_cfg<64, 64, 64, 64, AKS, BKS, EPI, false>(a, n, stream);
    case GEMM_TILE_128x128_DEALT: return launch_cfg<128, 128, 128, 128, AKS, BKS, EPI, false>(a, n, stream);
    default:                return launch_cfg<128, 128, 64, 64, AKS, BKS, EPI, false>(a, n, stream);
  }
}

// products held back for the next launch (GemmArgs::join)
thread_local GemmArgs g_held[GEMM_GROUP];
thread_local int g_nheld = 0;

}  // namespace

hipError_t gemm_launch(int layout, int epi, const GemmArgs& a0, int tile_cfg, hipStream_t stream) {
  const GemmArgs* a = &a0;
  int n = 1;
  if (a0.join || g_nheld) {
    if (layout != GEMM_TN || epi != EPI_ACC_F32) { g_nheld = 0; return hipErrorInvalidValue; }
    GemmArgs* last = g_nheld ? &g_held[g_nheld - 1] : nullptr;
    if (last && last->C == a0.C) {      // the next rows of the same product
      if (static_cast<const char*>(last->A) + (long)last->K * last->lda * 2 != a0.A ||
          static_cast<const char*>(last->B) + (long)last->K * last->ldb * 2 != a0.B || !a0.beta) { g_nheld = 0; return hipErrorInvalidValue; }
      last->K += a0.K;
    } else {
      if (g_nheld == GEMM_GROUP) { g_nheld = 0; return hipErrorInvalidValue; }
      g_held[g_nheld++] = a0;
    }
    if (a0.join) return hipSuccess;
    a = g_held; n = g_nheld; g_nheld = 0;
  }
  if (tile_cfg < 0) tile_cfg = gemm_pick_form(a, n, epi, a->concurrency);
  if (a0.tail) {      // a norm that is held has to fit the launch: four waves or more a workgroup, one range, the kernel's form of it
    const NormBwdArgs& norm = t_tail.norm;
    const bool norm_fits = norm.rows == 0 || (a->splits <= 1 && norm.h <= HeldTail::MAX_H && !norm.part_dres && !norm_streams(norm.rows, norm.h));
    if (!t_tail.open || t_tail.stream != stream || layout != GEMM_TN || !norm_fits) {
      t_tail.open = false;
      return hipErrorInvalidValue;
    }
  }
  if (layout == GEMM_NN) {
    switch (epi) {
      case EPI_STORE:     return launch_layout<false, true, EPI_STORE>(a, n, tile_cfg, stream);
      case EPI_BIAS_GELU: return launch_layout<false, true, EPI_BIAS_GELU>(a, n, tile_cfg, stream);
      case EPI_SWIGLU:    return launch_layout<false, true, EPI_SWIGLU>(a, n, tile_cfg, stream);
      case EPI_ROPE:      return launch_layout<false, true, EPI_ROPE>(a, n, tile_cfg, stream);
      case EPI_RESID:     return launch_layout<false, true, EPI_RESID>(a, n, tile_cfg, stream);
      default: return hipErrorInvalidValue;
    }
  } else if (layout == GEMM_NT) {
    switch (epi) {
      case EPI_STORE:   return launch_layout<false, false, EPI_STORE>(a, n, tile_cfg, stream);
      case EPI_DGELU:   return launch_layout<false, false, EPI_DGELU>(a, n, tile_cfg, stream);
      case EPI_DSWIGLU: return launch_layout<false, false, EPI_DSWIGLU>(a, n, tile_cfg, stream);
      default: return hipErrorInvalidValue;
    }
  } else if (layout == GEMM_TN) {
    if (epi == EPI_ACC_F32) return launch_layout<true, true, EPI_ACC_F32>(a, n, tile_cfg, stream);
    return hipErrorInvalidValue;
  }
  return hipErrorInvalidValue;
}
