// Which form the launchers pick for given sizes, from the rules in csrc/gemm.h and csrc/attention.h alone (no GPU, no
// library).  Reads one question per line and answers each with one number:
//   gemm <epilogue> <M> <N> <K> <concurrency> <beside> [<adds>]   GemmTile of one product (SwiGLU: N gate columns)
//   joined <K> <concurrency> <beside> <ranges> <M N> x 4 [<adds>]   GemmTile of four weight gradients in one launch
//   output <M> <N> <K>                                    1: the block output in the product's epilogue, 0: a pass
//   attention <backward> <batch> <seq> <heads>            1: 32 positions per workgroup, 0: 128
//   serial <head_dim> <batch> <seq> <heads>               1: the 128-position forward takes a tile's parts one after the other
//   walk <seq> <ld> <head_dim> <tiles>                    the furthest byte of a [seq, ld] matrix that the attention forward's views of
//                                                         one head and that many tiles (and the two asked for ahead) reach, or -1 where
//                                                         a view is before the matrix
//   ranges <tiles> <depth> <floats>                       contraction ranges of joined weight gradients
#include <cstdio>
#include <cstring>

#include "../paper_2409_15241_amd/csrc/attention.h"
#include "../paper_2409_15241_amd/csrc/gemm.h"

int main() {
  char line[256], what[32];
  long v[13] = {};
  while (std::fgets(line, sizeof(line), stdin)) {
    const int n = std::sscanf(line, "%31s %ld %ld %ld %ld %ld %ld %ld %ld %ld %ld %ld %ld %ld", what, v, v + 1, v + 2, v + 3, v + 4, v + 5, v + 6, v + 7,
                              v + 8, v + 9, v + 10, v + 11, v + 12);
    if ((n == 7 || n == 8) && !std::strcmp(what, "gemm")) {
      GemmArgs a{};
      a.M = (int)v[1]; a.N = a.n_split = (int)v[2]; a.K = (int)v[3]; a.beside = (int)v[5]; a.beta = n == 8 ? (int)v[6] : 0;
      std::printf("%d\n", gemm_pick_form(&a, 1, (int)v[0], (int)v[4]));
    } else if ((n == 13 || n == 14) && !std::strcmp(what, "joined")) {
      GemmArgs a[GEMM_GROUP] = {};
      for (int i = 0; i < GEMM_GROUP; ++i) {
        a[i].M = (int)v[4 + 2 * i]; a[i].N = (int)v[5 + 2 * i]; a[i].K = (int)v[0]; a[i].beside = (int)v[2]; a[i].splits = (int)v[3]; a[i].beta = n == 14 ? (int)v[12] : 0;
      }
      std::printf("%d\n", gemm_pick_form(a, GEMM_GROUP, EPI_ACC_F32, (int)v[1]));
    } else if (n == 4 && !std::strcmp(what, "output")) {
      std::printf("%d\n", gemm_forms_output((int)v[0], (int)v[1], (int)v[2]) ? 1 : 0);
    } else if (n == 5 && !std::strcmp(what, "attention")) {
      AttnArgs a{};
      a.batch = (int)v[1]; a.seq = (int)v[2]; a.heads = (int)v[3];
      std::printf("%d\n", attention_split_pays(a, v[0] != 0) ? 1 : 0);
    } else if (n == 5 && !std::strcmp(what, "serial")) {
      AttnArgs a{};
      a.head_dim = (int)v[0]; a.batch = (int)v[1]; a.seq = (int)v[2]; a.heads = (int)v[3];
      std::printf("%d\n", attention_fwd_serial(a) ? 1 : 0);
    } else if (n == 5 && !std::strcmp(what, "walk")) {
      const int tile = attention_tile_bytes(v[1]), rows = (int)(v[3] * 64 < v[0] ? v[3] * 64 : v[0]);
      long at = 0, furthest = 0;
      int left = attention_view_bytes(rows, (int)v[1], (int)v[2]);
      bool before = false;
      for (long k = 0; k < v[3] + 2; ++k, at += tile, left = attention_left_behind(left, tile)) {
        if (left > 0) furthest = at + left > furthest ? at + left : furthest;
        before |= left > 0 && at < 0;
      }
      std::printf("%ld\n", before ? -1L : furthest);
    } else if (n == 4 && !std::strcmp(what, "ranges")) {
      std::printf("%d\n", gemm_wgrad_splits((int)v[0], (int)v[1], v[2]));
    } else {
      return 1;
    }
  }
  return 0;
}
