// Internal launcher interface of the bf16 MFMA GEMM (see gemm.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <cmath>

enum GemmLayout { GEMM_NN = 0, GEMM_NT = 1, GEMM_TN = 2 };
enum GemmEpilogue {
  EPI_STORE = 0,      // C = bf16(acc + bias)                      bias optional
  EPI_BIAS_GELU = 1,  // aux = bf16(acc + bias); C = bf16(GeLU(acc + bias))
  EPI_SWIGLU = 2,     // aux[:, n] = gate, aux[:, n_split + n] = up; C[:, n] = silu(gate) * up
  EPI_DGELU = 3,      // C = bf16(acc * GeLU'(aux))
  EPI_DSWIGLU = 4,    // C[:, n] = acc * up * silu'(gate); C[:, n_split + n] = acc * silu(gate)
  EPI_ACC_F32 = 5,    // C(fp32) = acc (+ C if beta)
  EPI_ROPE = 6,       // C = bf16(acc) with the rotary embedding applied to columns below rope_cols (heads of rope_d columns)
};
enum GemmTile { GEMM_TILE_128x128 = 0, GEMM_TILE_256x128 = 1, GEMM_TILE_256x256 = 2, GEMM_TILE_128x256 = 3,
                GEMM_TILE_64x64 = 4, GEMM_TILE_128x128_DEALT = 5 };

constexpr int GEMM_BK = 64;      // contraction elements per operand tile

struct GemmArgs {
  const void* A; const void* B; void* C;
  long lda, ldb, ldc;
  int M, N, K;
  const void* bias;      // bf16 [N] or null
  void* aux; long ldaux; // epilogue side tensor (read or written, see GemmEpilogue)
  int n_split;           // SwiGLU: number of gate (= up) columns
  int beta;              // EPI_ACC_F32: 1 = accumulate into C
  int rope_d, rope_seq, rope_cols;   // EPI_ROPE: head width (64 or 128), sequence length (position = row % seq), rotated columns
  float rope_log2_base;
  int gelu_tanh;
  int concurrency;       // launches of similar size expected in flight at once (other streams); 0 = 1
  int beside;            // 1: meant to share the chip with other launches, so not in a dealt form, which takes all of it
  int splits;            // joined weight gradients: contraction ranges, each summed into its own part of split_ws (0 or 1: one)
  float* split_ws;       // splits * (sum of M * N of the joined products) floats
  int join;              // EPI_ACC_F32: 1 = hold this product back, it is launched together with the next call's (see gemm_launch)
  int tiles_m, tiles_n;  // filled by the launcher
  int group_m;           // filled by the launcher: tile rows per band of the tile order
  long a_bytes, b_bytes; // extent of the A / B views in bytes, filled by the launcher
};

// tile_cfg < 0: pick by shape.  Enqueues on `stream`; returns the launch status.
// Products with `join` set are held back (per thread) until the next call without it, which must follow on the same
// stream: at most GEMM_GROUP weight gradients then go out as one launch.  A product into the matrix of the one before it,
// over the rows that follow it (the next slice of the batch), continues that product's contraction.
constexpr int GEMM_GROUP = 4;

// Contraction ranges for weight gradients that are launched together and have the chip to themselves: `tiles` tiles of
// 256x256, `depth` deep, `floats` values in all.  A launch of 160 such tiles leaves 96 of 256 compute units idle for as
// long as its contraction is deep; cut into ranges it is rounds of shorter tiles, for partial sums that are written and
// read once each.  (us per tile and per byte as in the tile choice of gemm.hip.)
constexpr int GEMM_MAX_SPLITS = 6;
inline int gemm_wgrad_splits(int tiles, int depth, long floats) {
  const int it = (depth + 63) / 64;
  auto rounds = [&](int s) { return (tiles * s + 255) / 256 * (13.0 + 1.2 * ((it + s - 1) / s)); };
  double cost = rounds(1);
  if (const double t64 = (tiles + 15) / 16 * (1.8 + 1.4 * ((it + 7) / 8)); t64 < cost) cost = t64;              // in 64x64 tiles
  if (const double t128 = (tiles / 128) * (6 + 0.8 * it) + 3.4 + 0.47 * it; t128 < cost) cost = t128;           // in 128x128 tiles
  cost *= 0.9;
  int best = 1;
  for (int s = 2; s <= GEMM_MAX_SPLITS; ++s) {
    const double c = rounds(s) + 4.0 + 2.0 * s * floats * 4 / 5e6;
    if (c < cost) { cost = c; best = s; }
  }
  return best;
}
// Time of a launch that has the chip to itself = 3 us + rounds of tiles on 256 compute units x time of a tile; time of a
// tile = what its start and its epilogue take + what 64 elements of the contraction take (us; fitted to 77 shapes of 128 to
// 4096 rows, 640 to 7168 columns, 256 to 16384 deep).  128x128 tiles run two to a unit; one that is alone is faster, less
// so on long rows, whose loads come from further away.
// A launch beside three or more others of its size pays for the work and the padding of ragged edges only, the other
// launches fill the rest of its last round; beside one other, half way between.
// The dealt forms (gemm_split_body of gemm.hip) sum in another order than the rest: whether they are taken is decided as if nothing
// ran beside the launch, so that no bit of a result depends on the stream pool, and products meant to run beside others
// never take them.  They win where the other shapes leave most of the chip idle: 512 rows x 1920 columns x 5120 deep
// 41 -> 19 us, 240 x 2688 x 7168 82 -> 31, 1024 x 2688 x 7168 79 -> 57, 2048 x 1920 x 5120 55 -> 46, 256 x 1024 x 1024
// 10.0 -> 6.5; about 3000 deep the plain 128x128 tile meets the dealt one.
inline int gemm_pick_form(const GemmArgs* products, int n, int epi, int concurrency) {
  if (concurrency < 1) concurrency = 1;
  const bool swiglu = epi == EPI_SWIGLU;
  struct Cand { int id, bm, bn; double fixed, per64; };
  static const Cand cands[] = {{GEMM_TILE_256x256, 256, 256, 8.0, 1.06}, {GEMM_TILE_256x128, 256, 128, 4.0, 0.70},
                               {GEMM_TILE_128x256, 128, 256, 4.0, 0.73}, {GEMM_TILE_128x128, 128, 128, 1.5, 0.40}};
  // what the epilogue takes beyond storing bf16 sums, for 256x256 values: activations (vector ALUs), wider results
  const double extra = epi == EPI_BIAS_GELU ? 6.0 : epi == EPI_SWIGLU ? 5.0 : epi == EPI_DGELU ? 8.0 : epi == EPI_DSWIGLU ? 12.0 :
                       epi == EPI_ACC_F32 ? 5.0 : epi == EPI_ROPE ? 4.0 : 0.0;
  const int splits = products[0].splits > 1 ? products[0].splits : 1;
  auto tiles_of = [&](int bm, int bn) {
    double t = 0;
    for (int i = 0; i < n; ++i) {
      const int N = swiglu ? 2 * products[i].n_split : products[i].N;
      t += (double)((products[i].M + bm - 1) / bm) * ((N + bn - 1) / bn);
    }
    return t * splits;
  };
  const int it = ((products[0].K + GEMM_BK - 1) / GEMM_BK + splits - 1) / splits;      // a group's products share the contraction
  int best = GEMM_TILE_128x128;
  double best_cost = 1e30, best_alone = 1e30;
  for (const Cand& c : cands) {
    const double tiles = tiles_of(c.bm, c.bn), fixed = c.fixed + extra * c.bm * c.bn / 65536, unit = fixed + c.per64 * it;
    double alone;
    if (c.id == GEMM_TILE_128x128) {
      const double lone = fixed + 0.5 + 0.47 * (it < 40 ? it : 40) + 0.66 * (it < 40 ? 0 : it - 40), full = floor(tiles / 512), rest = tiles - 512 * full;
      alone = full * 2 * unit + (rest == 0 ? 0.0 : rest <= 256 ? lone : 2 * unit);
    } else {
      alone = ceil(tiles / 256) * unit;
    }
    best_alone = alone < best_alone ? alone : best_alone;
    // a launch of few tiles is a long serial kernel on its stream, and the other launches in flight do not always fill
    // the chip beside it: it is charged for leaving more than three eighths of its share of the chip unused
    const double share = 160.0 / concurrency;
    const double shared = (tiles < share ? share : tiles) / 256 * unit;
    const double cost = concurrency == 1 ? alone : concurrency == 2 ? 0.5 * (alone + shared) : shared;
    if (cost < best_cost * 0.999) { best_cost = cost; best = c.id; }
  }
  if (products[0].beside || splits > 1) return best;
  const double dealt64 = ceil(tiles_of(64, 64) / 256) * (1.8 + (epi == EPI_SWIGLU ? 0.4 : 0.15) * extra + 1.4 * ((it + 7) / 8));
  const double dealt128 = ceil(tiles_of(128, 128) / 256) * (7.0 + 0.3 * extra + 0.40 * it);
  if (3 + (dealt64 < dealt128 ? dealt64 : dealt128) >= 0.95 * (3 + best_alone)) return best;
  return dealt64 < dealt128 ? GEMM_TILE_64x64 : GEMM_TILE_128x128_DEALT;
}

hipError_t gemm_launch(int layout, int epi, const GemmArgs& a, int tile_cfg, hipStream_t stream);
