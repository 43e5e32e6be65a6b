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
  EPI_RESID = 7,      // C = bf16(acc); out2 = bf16(aux + C + add2 + bias)   add2, bias optional: the block output with its last partial sum
};
enum GemmTile { GEMM_TILE_128x128 = 0, GEMM_TILE_256x128 = 1, GEMM_TILE_256x256 = 2, GEMM_TILE_128x256 = 3,
                GEMM_TILE_64x64 = 4, GEMM_TILE_128x128_DEALT = 5,
                GEMM_TILE_256x192 = 6, GEMM_TILE_192x256 = 7, GEMM_TILE_256x320 = 8, GEMM_TILE_320x256 = 9 };

constexpr int GEMM_BK = 64;      // contraction elements per operand tile

struct GemmArgs {
  const void* A; const void* B; void* C;
  long lda, ldb, ldc;
  int M, N, K;
  const void* bias;      // bf16 [N] or null
  void* aux; long ldaux; // epilogue side tensor (read or written, see GemmEpilogue)
  const void* add2; void* out2;      // EPI_RESID: bf16, rows of ldaux
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
  int tail;              // joined weight gradients: 1 = with what t_tail of norm.h holds for their stream; filled in by the launcher for the kernels
  int tiles_m, tiles_n;  // filled by the launcher
  int group_m;           // filled by the launcher: tile rows per band of the tile order
  long a_bytes, b_bytes; // extent of the A / B views in bytes, filled by the launcher
};

// tile_cfg < 0: pick by shape.  Enqueues on `stream`; returns the launch status.
// Products with `join` set are held back (per thread) until the next call without it, which must follow on the same
// stream: at most GEMM_GROUP weight gradients then go out as one launch.  A product into the matrix of the one before it,
// over the rows that follow it (the next slice of the batch), continues that product's contraction.
constexpr int GEMM_GROUP = 4;

// Time of a launch that has the chip to itself = 3 us + rounds of tiles on 256 compute units x time of a tile; time of a tile
// = what its start and its epilogue take (fixed) + what 64 elements of the contraction take: `full` where the round fills the
// chip, whose clocks then fall to what its power allows, `lone` where few compute units are at work, in proportion between
// (us; fitted to timings of 921 products of shards like the library's, 128 to 32768 rows, 64 to 28672 columns, 80 to 8192
// deep, operands out of the caches; 128x256 was the fastest for one of them and is not looked at.  Of 1274 others, drawn
// afterwards, the form picked is the fastest at the median, within 5 % of it for nine tenths and within 17 % for 99 of 100).
// Forms of 192 and 320 rows or columns are there for the last round: 16384 x 1280 x 2560 is 320 tiles of 256x256, the second
// round a quarter full, or 256 of 256x320 (108 -> 79 us; 8192 x 2560 x 5120 206 -> 147; 8192 x 2688 x 7168, 352 tiles or 448 of
// 256x192, 274 -> 227).  A pair of columns that must meet in a lane rules out those with wave tiles of 96 or 160 columns.
// adds: what adding to the fp32 values that C holds takes beyond overwriting them, for 256x256 values.  12 or 13 is reading them
// at the rate of memory; some forms measure twice that; 128x128 tiles pay less, one of the two workgroups of a compute unit
// loading while the other multiplies.  (Four weight gradients in one launch, adding, 71 such blocks of 64 to 4096 tokens: the
// form picked is 0.5 % above the fastest on the mean and 13 % at most, without this term 17 and 56 %.  192 tokens of a 6144-wide
// shard 150 us in 192x256, 110 in 128x128; 512 of a 1536-wide one 31 in 256x128, 23 in 128x128.)
struct GemmForm { int id, bm, bn; double fixed, lone, full, adds; };
constexpr GemmForm GEMM_FORMS[] = {
  {GEMM_TILE_256x256, 256, 256, 6.1, 1.17, 1.335, 12}, {GEMM_TILE_256x320, 256, 320, 9.5, 1.46, 1.85, 12}, {GEMM_TILE_320x256, 320, 256, 7.6, 1.49, 2.00, 22},
  {GEMM_TILE_256x192, 256, 192, 4.8, 0.86, 1.19, 13}, {GEMM_TILE_192x256, 192, 256, 4.3, 0.89, 1.27, 20}, {GEMM_TILE_256x128, 256, 128, 3.4, 0.57, 0.90, 24},
  {GEMM_TILE_128x128, 128, 128, 2.1, 0.39, 0.47, 8}};
// what the epilogue takes beyond storing bf16 sums, for 256x256 values: activations (vector ALUs), wider results
inline double gemm_epilogue_time(int epi) {
  return epi == EPI_BIAS_GELU ? 5.9 : epi == EPI_SWIGLU ? 8.2 : epi == EPI_DGELU ? 8.9 : epi == EPI_DSWIGLU ? 10.6 :
         epi == EPI_ACC_F32 ? 5.0 : epi == EPI_ROPE ? 4.0 : epi == EPI_RESID ? 8.0 : 0.0;
}
inline bool gemm_form_takes(const GemmForm& f, int epi) {
  if (epi == EPI_RESID) return f.bn != 320;                    // see gemm_forms_output
  return (epi != EPI_SWIGLU && epi != EPI_ROPE) || (f.bn != 192 && f.bn != 320);
}
// tiles of contraction `it` x 64 deep; 128x128 tiles run two to a compute unit
inline double gemm_form_time(const GemmForm& f, double tiles, int it, int epi, bool adds = false) {
  const double fixed = f.fixed + (gemm_epilogue_time(epi) + (adds ? f.adds : 0.0)) * f.bm * f.bn / 65536;
  if (f.id == GEMM_TILE_128x128) {
    const double rounds = floor(tiles / 512), rest = tiles - 512 * rounds, share = f.full * rest / 512;
    return 3 + rounds * 2 * (fixed + f.full * it) + (rest == 0 ? 0.0 : rest <= 256 ? fixed - 1.1 + 0.503 * (it < 40 ? it : 40) + (it < 40 ? 0.0 : 0.80 * (it - 40)) : 2 * (fixed + (f.lone > share ? f.lone : share) * it));
  }
  const double rounds = floor(tiles / 256), rest = tiles - 256 * rounds, share = f.full * rest / 256;
  return 3 + rounds * (fixed + f.full * it) + (rest == 0 ? 0.0 : fixed + (f.lone > share ? f.lone : share) * it);
}

// Contraction ranges for weight gradients that are launched together and have the chip to themselves: `tiles` tiles of
// 256x256, `depth` deep, `floats` values in all.  A launch of 160 such tiles leaves 96 of 256 compute units idle for as
// long as its contraction is deep; cut into ranges it is rounds of shorter tiles, for partial sums that are written and
// read once each.  (13 + 1.2 us per 64 deep and tile, 5 TB/s for the sums: coarser figures than GEMM_FORMS, of 256x256 tiles
// alone.  Of ten blocks timed with 1 to 6 ranges the rule is within 1.3 % of the best for nine; 24000 tokens of a 1536-wide
// shard, 114 tiles, take 1642 us with the one range that it gives and 1599 with two.  16384 tokens of a 512-wide block, 48 tiles:
// 690 us with one range, 659 with the rule's five; 2.7B with 32768 tokens, 160 tiles, 2710 and 2672 with three.)
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

// The form of a launch of n products.  A launch beside three or more others of its size pays for the work and the padding of
// ragged edges only, the other launches fill the rest of its last round; beside one other, a third of the way from there to a launch alone.
// The dealt forms (gemm_split_body of gemm.hip) sum in another order than the rest: whether they are taken is decided as if nothing
// ran beside the launch, so that no bit of a result depends on the stream pool, and products meant to run beside others
// never take them.  The product that forms the block output in its epilogue takes them where the plain product does, which
// a stack runs in its place in all blocks but the last: a block's sums are the same alone and in a stack.
// They win where the other shapes leave most of the chip idle: 512 rows x 1920 columns x 5120 deep
// 41 -> 19 us, 240 x 2688 x 7168 82 -> 31, 1024 x 2688 x 7168 79 -> 57, 2048 x 1920 x 5120 55 -> 46, 256 x 1024 x 1024
// 10.0 -> 6.5; about 3000 deep the plain 128x128 tile meets the dealt one.
inline int gemm_pick_form(const GemmArgs* products, int n, int epi, int concurrency) {
  if (concurrency < 1) concurrency = 1;
  if (epi == EPI_RESID) {
    const int plain = gemm_pick_form(products, n, EPI_STORE, concurrency);
    if (plain == GEMM_TILE_64x64 || plain == GEMM_TILE_128x128_DEALT) return plain;
  }
  const int splits = products[0].splits > 1 ? products[0].splits : 1;
  auto tiles_of = [&](int bm, int bn) {
    double t = 0;
    for (int i = 0; i < n; ++i) {
      const int N = epi == EPI_SWIGLU ? 2 * products[i].n_split : products[i].N;
      t += (double)((products[i].M + bm - 1) / bm) * ((N + bn - 1) / bn);
    }
    return t * splits;
  };
  const int it = ((products[0].K + GEMM_BK - 1) / GEMM_BK + splits - 1) / splits;      // a group's products share the contraction
  const double extra = gemm_epilogue_time(epi);
  const bool adds = epi == EPI_ACC_F32 && products[0].beta && splits == 1;      // (ranges write sums of their own)
  int best = GEMM_TILE_128x128;
  double best_cost = 1e30, best_alone = 1e30;
  for (const GemmForm& f : GEMM_FORMS) {
    if (!gemm_form_takes(f, epi)) continue;
    const double tiles = tiles_of(f.bm, f.bn), over = gemm_form_time(f, tiles, it, epi), alone = adds ? gemm_form_time(f, tiles, it, epi, true) : over;
    best_alone = over < best_alone ? over : best_alone;      // whether a contraction is dealt does not depend on what C holds either
    // a launch of few tiles is a long serial kernel on its stream, and the other launches in flight do not always fill
    // the chip beside it: it is charged for leaving more than three eighths of its share of the chip unused
    const double share = 160.0 / concurrency;
    const double shared = 3 + (tiles < share ? share : tiles) / 256 * (f.fixed + (extra + (adds ? f.adds : 0.0)) * f.bm * f.bn / 65536 + f.full * it);
    const double cost = concurrency == 1 ? alone : concurrency == 2 ? 0.35 * alone + 0.65 * shared : shared;
    if (cost < best_cost * 0.999) { best_cost = cost; best = f.id; }
  }
  if (products[0].beside || splits > 1 || epi == EPI_RESID) return best;
  const double dealt64 = 1.7 + ceil(tiles_of(64, 64) / 256) * (1.9 + (epi == EPI_SWIGLU ? 0.23 : 0.07) * extra + 1.68 * ((it + 7) / 8));
  const double dealt128 = 3 + ceil(tiles_of(128, 128) / 256) * (7.0 + 0.36 * extra + 0.403 * it);
  if ((dealt64 < dealt128 ? dealt64 : dealt128) >= best_alone) return best;
  return dealt64 < dealt128 ? GEMM_TILE_64x64 : GEMM_TILE_128x128_DEALT;
}

// Whether the product that completes a block's sums forms the block output in its epilogue (EPI_RESID), or a pass over memory
// does behind the plain product.  The epilogue moves four rows of bf16 where a plain one stores one: it saves a launch and
// the sums' way through memory, but runs at a tile's end, with the matrix cores idle.  That pays except where the plain
// product takes 256x320 tiles: one round of those or little more has the longest epilogues, and the last 32 columns of a
// 160-wide wave tile move in half lines.  (Forward of a block, us, pass and epilogue.  256x320: 2.7B with 8192 tokens 281
// and 288, 13B with 4096 391 and 397, Llama-2 13B with 4096 385 and 390, 2.7B with 16384 520 and 525.  Other tiles: 2.7B
// with 4096 160 and 156, with 6018 228 and 225, 13B with 1024 156 and 151, with 2048 237 and 235, Llama-2 7B with 2 x 4096
// 599 and 587, a 1024-wide block with 16384 329 and 324; 6.7B with 4096 and 30B with 2048 are level, a 3072-wide one with
// 4096 is 1 % slower.)
inline bool gemm_forms_output(int M, int N, int K) {
  GemmArgs a{};
  a.M = M; a.N = N; a.K = K;
  return gemm_pick_form(&a, 1, EPI_STORE, 1) != GEMM_TILE_256x320;
}

hipError_t gemm_launch(int layout, int epi, const GemmArgs& a, int tile_cfg, hipStream_t stream);
