// Internal launcher interface of the bf16 MFMA GEMM (see gemm.hip).
#pragma once
#include <hip/hip_runtime.h>
#include <type_traits>

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
hipError_t gemm_launch(int layout, int epi, const GemmArgs& a, int tile_cfg, hipStream_t stream);
