// Internal launcher interface of the attention kernels (see attention.hip).
#pragma once
#include <hip/hip_runtime.h>

struct AttnArgs {
  const void* qkv;     // bf16 [batch*seq, ld]: q | k | v column blocks, heads contiguous inside a block
  long ld;
  void* ctx;           // bf16 [batch*seq, ld_ctx]: forward output / backward input
  long ld_ctx;
  const void* dctx;    // bf16 [batch*seq, ld_ctx] (backward)
  float* lse;          // fp32 [batch, heads, seq]
  float* dot;          // fp32 [batch, heads, seq]: rowsum(dctx * ctx) (backward scratch)
  void* dqkv;          // bf16 [batch*seq, ld] (backward output)
  int batch, seq, heads, head_dim;
  float scale;         // 1 / sqrt(head_dim)
  int rope;            // backward: q and k of qkv carry the rotary embedding; dq and dk are turned back before the store
  float rope_log2_base;
};

// Whether the form for few workgroups (32 positions each, see attention.hip) is the faster one, from the time of either on
// an otherwise idle chip (us): the longest workgroup's chain against the split form's start, end and rounds of workgroups.
// Forward / backward, heads of 128: 4 x 704 positions, one head 14.0 -> 12.1 / 30.7 -> 18.6; 812, seven heads 16.1 -> 14.6 /
// 35.0 -> 24.4; 4096, two heads 60 -> 42 / 118 -> 67; the two forms meet at 3 x 1024, four heads, backward (42.2 and 41.2).
// The constants were fitted before either 128-position form ran its softmax under its MFMAs, which moved where they
// meet: forward, heads of 128, 4 x 512, five heads 13.0 in the form not taken, 14.2 in the one that is, 8 x 512, four heads 13.1 and 16.4,
// 8 x 384, five heads 11.2 and 15.3, where 3 x 1024, four heads is right with 20.0 and 18.6; backward 2 x 2048, four heads 70.1 and 75.5.
// They have not been fitted again since.
inline bool attention_split_pays(const AttnArgs& a, bool backward) {
  const int wgs = (a.seq + 127) / 128 * a.heads * a.batch, steps = (a.seq + 63) / 64;
  if (wgs > 128) return false;
  const double at_once = backward ? wgs / 32.0 : wgs / 96.0, rounds = at_once > 1.0 ? at_once : 1.0;
  if (backward) return 11 + rounds * (5 + 1.45 * a.seq / 256) < 0.95 * (14 + 2.15 * steps);
  return 4.5 + rounds * (1.5 + 1.1 * a.seq / 128) < 0.95 * (5 + 1.17 * steps);
}

// Whether the 128-position forward takes each tile's scores, softmax and output one after the other (attn_fwd_serial_kernel) and not two
// tiles at once (attn_fwd_kernel); both give the same bits.  Two at once needs 204 registers for heads of 64, so that a compute unit takes
// two workgroups where it takes three of the serial form: of 512 < n <= 768 workgroups the last wait for a second round, and in
// several rounds three that alternate hide a tile's chain as well as two tiles a wave (us, two at once / serial: 256 positions x 308 heads
// 14.1 / 11.8, 64 x 640 7.5 / 5.8, 1024 x 256 62.0 / 55.1, 4096 x 64 171 / 166; up to 512 workgroups 4096 x 8 48.9 / 59.7, 704 x 64
// 12.3 / 13.9, but of few tiles, two workgroups to a compute unit, 256 x 256 9.7 / 8.9, 192 x 160 7.0 / 6.8; of 769 to 1024, two rounds either way, 192 x 400 12.3 / 13.4, 1024 x 128 28.4 / 29.5, but 512 x 200 19.1 / 17.3).  Heads of
// 80 and 128 take two workgroups in either form, and one tile leaves nothing to overlap (64 positions: 256 heads of 64 4.4 / 4.2, of 80
// 4.9 / 4.7, 512 of 128 8.3 / 7.8); heads of 128 of two tiles, two workgroups to some compute units, 128 x 308 11.5 / 10.8, 100 x 400
// 10.7 / 10.1, but x 256 level and x 160 6.9 / 7.2.  All with the operands in the caches, as the QKV product in front leaves them; out
// of them heads of 128 of two tiles would be the other way round, 128 x 308 16.1 / 17.4.
inline bool attention_fwd_serial(const AttnArgs& a) {
  const long wgs = (long)((a.seq + 127) / 128) * a.heads * a.batch;
  if (a.seq <= 64) return true;
  if (a.head_dim == 64) return wgs > 512 ? wgs <= 768 || wgs > 1024 : wgs > 256 && a.seq <= 256;
  return a.head_dim == 128 && a.seq <= 128 && wgs > 256 && wgs <= 512;
}

// Whether the backward of the form for few workgroups forms D = rowsum(dctx * ctx) itself, where a wave has two tiles of 32 queries or fewer: it saves a dependent launch
// and costs 0.85 us a tile of a wave's chain (16-byte loads of 32 rows, which nothing else covers).  Backward with the launch and
// without, us: 2 x 128 positions, two heads of 64 7.8 and 6.0, 2 x 200, two of 128 12.1 and 10.7, 4 x 256 12.4 and 11.5; 2 x 512, four heads
// 15.3 and 16.3, 2 x 1024, two 20.7 and 25.4, 4096, two 62 and 90.
inline bool attention_owns_d(int seq) { return seq <= 256; }

// How the 128-position forward walks a view of K or V: `left` bytes from a tile's first row to the end of the last row needed, tiles
// of 64 rows of `ld` values.  A matrix is smaller than 2 GiB, 64 rows of it need not be (few rows of more than 2^24 values): such a tile
// is the last, whatever its size.  No sum or difference here leaves 31 bits.
constexpr int attention_view_bytes(int rows, int ld, int head_dim) { return ((rows - 1) * ld + head_dim) * 2; }
constexpr int attention_tile_bytes(long ld) { return ld < 1L << 24 ? (int)(64 * ld * 2) : 0x7fffffff; }
constexpr int attention_left_behind(int left, int tile_bytes) { return left > tile_bytes ? left - tile_bytes : 0; }

hipError_t attention_fwd_launch(const AttnArgs& a, hipStream_t st);
hipError_t attention_bwd_launch(const AttnArgs& a, hipStream_t st);
