// How the matmuls of a pass are divided into workgroups: pure functions of the shape and of the number of rows.
#pragma once

#include "internal.hpp"

namespace ts {

inline int rows_pad_for(int rows) {
  if (rows <= 32) return 32;
  if (rows <= 64) return 64;
  if (rows <= 128) return 128;
  return 256;
}

struct SplitPlan {
  int kernel;   // GEMM_*
  int tile_n, n_tiles, n_splits, k_per_split;
};

inline int tiles_of(int n) { return (n + kGemmTileN - 1) / kGemmTileN; }
// 16-row blocks that the streaming kernel multiplies for a panel of up to 128 rows: 1 to 4, 6 or 8.
inline int row_blocks(int rows) { return rows <= 64 ? (rows + 15) / 16 : (rows <= 96 ? 6 : 8); }

// Tile widths that the streaming kernel is built in, by 16-row blocks of its tile.  QKV: whole rotation pairs.  The sums of
// squares of any 16 columns of a residual product stand for themselves.  The adapter's plain product: one width.  LM
// head: widths that the 128-column kernel does not take.  Accumulators of 128 x 128, for QKV also 96 columns over more than
// 64 rows, for gate + up 112, do not fit.  Gate + up in 112 columns makes one tile a CU of 28672 (us over 9 / 30 / 60 rows,
// 4096 deep): 112 columns 38.2 / 39.8 / 47.5, 96 51.9 / 57.0 / 70.9, 64 42.0 / 46.9 / 59.2, 48 48.5 / 58.0 / 77.7; of 24576 96 columns
// do (60 rows 43.0, 112 53.2, 64 56.9).  80 columns, one tile a CU of 20480, are not built.
constexpr bool stream_built(int epi, int tile_n, int rb) {
  if (rb < 1 || rb > 8 || rb == 5 || rb == 7) return false;
  if (epi == EPI_HEAD) return tile_n == 128 && rb <= 4;
  if (epi == EPI_PLAIN) return tile_n == 32;
  if (epi == EPI_SWIGLU) return tile_n == 32 || tile_n == 48 || tile_n == 64 || tile_n == 96 || (tile_n == 112 && rb <= 4);
  if (tile_n == 96) return epi == EPI_QKV && rb <= 4;
  return tile_n == 16 || tile_n == 32 || tile_n == 64 || (tile_n == 128 && rb <= 4);
}

// Tiles of three row blocks and more, in as many splits at least: the workgroups of a tile finish it together, a block of 16 rows
// each.  One workgroup with two blocks after another takes longer than the last to arrive with the whole tile (128 rows in 4 splits: 44.1 ->
// 44.9 us).  Tiles of two blocks, and two blocks by one workgroup in one round trip, have not been measured.
constexpr int kMeetBlocks = 3, kMaxStreamSplits = 16;   // a word of meet_splits has room for 16
constexpr bool tile_meets(int epi, int rb, int n_splits) {
  return epi != EPI_HEAD && epi != EPI_SWIGLU && rb >= kMeetBlocks && n_splits >= rb;
}

// Decomposition of one matmul over at most 128 rows into (column tile, k split) workgroups of the streaming
// kernel (gemm_stream.hpp): the tile width and the number of splits with the smallest estimated time.
//
// The estimate.  A workgroup takes 3 us to its first data.  It then draws its weights and its share of the
// activation panel, 2 bytes a column and 64 a row block and k step, at 45 (one row block) to 60 GB/s; the chip draws no
// more than 6.3 TB/s of weights.  Finishing a tile takes 0.012 us a row block and column, meeting the other splits
// 0.8 us more and 0.002 a split, row block and column: publish the partial tile, count, read all of them.  A tile whose workgroups
// finish it together (tile_meets) takes 1.2 us, 0.001 a row block and column, 0.0008 a split and column, 0.05 a split and 0.15 of
// its stream instead (the slowest one's lead).  So wide tiles draw less of the panel and narrow ones meet sooner.  256 workgroups at a time: one a CU, as most tiles fill it (16 and 32 columns
// over at most 32 rows would fit one to four times, by ring depth).  What it does not know: the ring's depth (launch_ring in
// gemm_stream.hpp), and the epilogues apart (QKV in wide tiles takes 1 to 4 us more than estimated).  Eight and more splits
// and more than 64 rows cost less than estimated.
//
// Estimated / measured, us (kernel times over cold weights; * chosen):
// By one workgroup:
//   4096 x 4096, 60 rows    32 x 2 16.8 / 17.0   64 x 4 15.5 / 16.5   128 x 8 23.5 / 18.4   16 x 1 23.4 / 18.3   32 x 1 26.4 / 21.2
//   4096 x 12288, 60 rows   64 x 4 28.6 / 31.6   128 x 8 34.1 / 30.9   32 x 2 38.6 / 36.4   64 x 2 47.2 / 44.8   32 x 1 70.1 / 58.1
//   6144 x 4096 (QKV), 60   96 x 4 19.5 / 23.3   64 x 2 21.0 / 22.3   128 x 4 22.8 / 24.7   96 x 2 25.2 / 26.6   32 x 1 26.4 / 23.7
//   24576 x 4096 (gate + up), 60   96* 39.6 / 43.0   112 41.1 / 53.2   48 56.4 / 56.5   64 61.5 / 56.9   32 76.1 / 67.0
//   2048 x 2048, 60 rows    32 x 4 9.1 / 8.9   16 x 2 9.7 / 9.7   32 x 2 11.3 / 10.8   64 x 8 12.6 / 10.8
//   2048 x 6144, 60 rows    32 x 4 14.6 / 14.0   64 x 8 15.9 / 15.2   16 x 2 19.6 / 17.1   32 x 2 22.2 / 19.7
//   2048 x 2048, 111 rows   32 x 4* 13.8 / 11.5   16 x 2 15.1 / 12.7   32 x 2 17.7 / 14.3   64 x 4 19.5 / 15.6
//   2048 x 6144, 111 rows   32 x 4 23.7 / 19.8   64 x 8 26.3 / 20.6   64 x 4 30.4 / 24.3   16 x 2 33.7 / 25.7
// All of the tile together:
//   4096 x 4096, 60 rows    64 x 4* 15.5 / 15.9   128 x 8 18.0 / 17.6
//   4096 x 12288, 60 rows   128 x 8* 30.0 / 28.1   128 x 7 31.8 / 30.1
//   6144 x 4096 (QKV), 60   96 x 4* 18.8 / 21.7   128 x 5 20.7 / 20.3
//   2048 x 2048, 60 rows    32 x 4* 9.4 / 8.8   64 x 8 10.2 / 11.2
//   2048 x 6144, 60 rows    64 x 8* 13.7 / 14.0   32 x 4, by one workgroup, 14.0
//   2048 x 6144, 111 rows   64 x 8* 21.1 / 16.7;   4096 x 2048 (QKV, norms), 111 rows   128 x 4 in two row groups 21.6 -> 16.4
//   1024 x 3072, 37 rows    32 x 8* 7.9 / 8.1   16 x 4 8.4 / 8.5;   1472 x 4032, 46 rows    32 x 5* 9.9 / 10.2   64 x 11 10.2 / 11.1
// Over few rows:
//   1024 x 2048, 9 rows     16 x 4* 5.2 / 6.4   32 x 4 5.9 / 6.6   16 x 2 6.2 / 6.6   32 x 2 7.2 / 7.3   16 x 1 7.6 / 6.5
//   1024 x 3072, 9 rows     16 x 4* 5.8 / 6.8   32 x 4 6.6 / 7.4   16 x 2 7.3 / 7.4   32 x 2 8.7 / 8.4   16 x 1 9.7 / 8.2
// Of the tilings measured the chosen one is the fastest or within 5 % of it, but for QKV 6144 x 4096 over 60 rows: 7 %, as the epilogue has no term.
inline SplitPlan plan_stream(int epi, int n_cols, int k, int rows, int head_dim, bool qk_norm) {
  const int steps = k / 32;
  SplitPlan best;
  best.kernel = GEMM_STREAM;
  best.k_per_split = k;
  best.n_splits = 1;
  best.tile_n = kGemmTileN;
  if (epi == EPI_HEAD) {   // widths that the 128-column kernel does not take
    best.n_tiles = tiles_of(n_cols);
    return best;
  }
  // Where q and k have a norm of their own a tile holds whole heads, over more than 64 rows in two groups of 64; other heads
  // of 128 are divided into rotation pairs by 96 columns too.
  const int widths[] = {16, 32, 48, 64, 96, 112, 128};
  double best_us = 1e30;
  for (int tn : widths) {
    int rb = row_blocks(rows), groups = 1;
    if (epi == EPI_QKV) {
      if ((qk_norm && tn < head_dim) || (tn == 96 && (qk_norm || head_dim != 128))) continue;
      if (tn == 128 && rb > 4) { rb = 4; groups = 2; }
    }
    if (!stream_built(epi, tn, rb)) continue;
    const int tiles = (n_cols + tn - 1) / tn;
    const double rate = rb == 1 ? 45e3 : 60e3, chip_us = 2.0 * n_cols * k / 6.3e6;
    for (int sp = 1; sp <= kMaxStreamSplits && sp <= steps && (sp == 1 || tiles * groups * sp <= 256); ++sp) {
      if (tile_meets(epi, rb, sp) && steps < 8 * sp) continue;   // a step for each of eight wavefronts; tiles of four are not told apart
      const int rounds = (tiles * groups * sp + 255) / 256;
      const double own_us = rounds * ((steps + sp - 1) / sp) * 32.0 * (2.0 * tn + 64.0 * rb) / rate;
      double us = 3.0 * rounds + (own_us > chip_us ? own_us : chip_us) + 0.012 * rb * tn;
      if (tile_meets(epi, rb, sp)) us += 1.2 + 0.001 * rb * tn + 0.0008 * sp * tn + 0.05 * sp + 0.15 * own_us;
      else if (sp > 1) us += 0.8 + 0.002 * sp * rb * tn;
      if (us < best_us) {
        best_us = us;
        best.tile_n = tn;
        best.n_tiles = tiles;
        best.n_splits = sp;
      }
      if (epi == EPI_SWIGLU) break;   // tiles enough: the kernel has no splits for it
    }
  }
  return best;
}
// Row groups of one plan: a QKV tile of 128 columns over more than 64 rows takes them in two groups of 64
inline int row_groups(int epi, const SplitPlan &p, int rows) { return epi == EPI_QKV && p.tile_n == 128 && rows > 64 ? 2 : 1; }
// The same of one launch
inline bool tiles_meet(const GemmArgs &g) {
  const bool groups = g.epi == EPI_QKV && g.tile_n == 128 && g.rows > 64;
  return g.kernel == GEMM_STREAM && tile_meets(g.epi, groups ? 4 : row_blocks(g.rows), g.n_splits);
}
// Tiles that meet at a counter: row groups have their own
inline int counted_tiles(int epi, const SplitPlan &p, int rows) { return p.n_tiles * row_groups(epi, p, rows); }
// Floats of its partial tiles
inline size_t stream_part_floats(int epi, const SplitPlan &p, int rows) {
  const int groups = row_groups(epi, p, rows), tile_rows = groups > 1 ? 64 : 16 * row_blocks(rows);
  return p.n_splits < 2 ? 0 : (size_t)p.n_splits * p.n_tiles * groups * tile_rows * p.tile_n;
}
// LM head over at most 128 rows: the 128-column kernel (kernels_gemm.hip) shares the activation panel among its
// wavefronts through LDS; it needs reductions of whole chunk pairs.  n_splits is the number of passes of a
// workgroup, n_tiles the entries that all of them leave: one pass each, but for more than 512 tiles (two workgroups a CU)
// over at most 32 rows, where 512 workgroups share the sub-tiles of 32 out.
constexpr int kHeadPlaces = 512;
inline int head_places(int n_cols) { return tiles_of(n_cols) < kHeadPlaces ? tiles_of(n_cols) : kHeadPlaces; }
inline int head_passes(int n_cols) {
  const int n_sub = (n_cols + 31) / 32, places = head_places(n_cols);
  return ((n_sub + places - 1) / places + 3) / 4;
}
inline SplitPlan plan_head(int n_cols, int k, int rows, int rows_pad) {
  if (k % (rows_pad == 32 ? 512 : 256) != 0) return plan_stream(EPI_HEAD, n_cols, k, rows, 0, false);
  SplitPlan p;
  p.kernel = GEMM_HEAD;
  p.tile_n = kGemmTileN;
  p.k_per_split = k;
  p.n_splits = rows_pad == 32 ? head_passes(n_cols) : 1;
  p.n_tiles = rows_pad == 32 ? head_places(n_cols) * p.n_splits : tiles_of(n_cols);
  return p;
}
// entries per row of the sums of squares that a matmul with tiles of tile_n columns leaves
inline int ss_tiles_of(int n, int tile_n) { return tile_n < kGemmTileN ? (n + tile_n - 1) / tile_n : tiles_of(n); }

constexpr int kWideRows = 128;   // rows of a workgroup of kernels_gemm_wide.hip
// Decomposition of one matmul over a panel of 256 rows, LM head also 128 (kernels_gemm_wide.hip): the tile width
// and the number of k splits with the smallest estimated time.  Fitted to products of 1024 to 4096 wide models: a 64-deep
// chunk takes a workgroup 1.65 us on a 128 x 256 tile and 1.0 us on a 128 x 128 tile, a workgroup about 6 us beside its
// chunks, one workgroup a CU (two of the 128-column tiles would fit); splitting costs 1.5 us (a second launch, but no epilogue in the first) and the
// partial tiles, written and read back at about 6.5 TB/s.  Estimated / measured, us, 240 rows: 6144 x 1024 in one split 22.0 / 21.7,
// two 19.4 / 18.8; 2048 x 6144 in four 34.1 / 33.6, eight 24.7 / 25.0; 4096 x 14336 (256 columns) in eight 64.0 / 65.2.
inline SplitPlan plan_wide(int epi, int n_cols, int k, int rows_pad, size_t max_part_floats) {
  const int kb = k / 64, n_rg = rows_pad / kWideRows;
  SplitPlan best;
  best.kernel = GEMM_WIDE;
  best.tile_n = 256;
  best.n_tiles = (n_cols + 255) / 256;
  best.n_splits = 1;
  best.k_per_split = k;
  if (epi == EPI_HEAD) return best;
  double best_us = 1e30;
  for (int tile_n = 256; tile_n >= 128; tile_n -= 128) {
    const int tiles = (n_cols + tile_n - 1) / tile_n;
    for (int s = 1; s <= 16 && s <= kb; ++s) {
      const size_t floats = (size_t)s * tiles_of(n_cols) * kGemmTileN * rows_pad;
      if (s > 1 && floats > max_part_floats) break;
      const int rounds = (tiles * n_rg * s + 255) / 256, chunks = (kb + s - 1) / s;
      const double us = rounds * (chunks * (tile_n == 256 ? 1.65 : 1.0) + 6.0) +
                        (s > 1 ? 1.5 + (double)floats * 8.0 / 6.5e6 : 0.0);
      if (us < best_us) {
        best_us = us;
        best.tile_n = tile_n;
        best.n_tiles = tiles;
        best.n_splits = s;
      }
    }
  }
  return best;
}
// Work items of a product in k splits are split * n_tiles + tile, at most a few hundred (kWidePartFloats).  item / n_tiles without a division:
constexpr uint32_t wide_tiles_inv(int n_tiles) { return n_tiles == 1 ? 0u : (uint32_t)((1ull << 32) / n_tiles + 1); }
constexpr int wide_split(int item, int n_tiles, uint32_t inv) { return n_tiles == 1 ? item : (int)((unsigned long long)(uint32_t)item * inv >> 32); }
// LM head of the wide kernel: one row group after the other, weights with the non-temporal hint, instead of the row groups of a tile
// side by side?  Where one group is all there is.  And where the workgroups are more than one round and the last group is short: behind
// full groups its workgroups, with a few rows to write out, fill the last round, which side by side is as long as the first.  us a pass of one
// layer, side by side -> apart: 132 rows, 36608 columns x 704 167.9 -> 129.3, x 4096 333.6 -> 288.8, 102400 x 4096 587 -> 544; 192 rows 175 -> 152, 347 ->
// 318, 603 -> 582; 208 rows, 36608 x 704 177 -> 167, x 4096 350 -> 334.  But then the weights come from memory again, once they are
// past the memory-side cache: 208 rows, 151936 x 2560 565 -> 581, 192 rows, 151936 x 4096 739 -> 756; 240 rows gain nothing.
constexpr bool wide_apart(int n_cols, int k, int rows) {
  const int groups = (rows + kWideRows - 1) / kWideRows, last = rows - (groups - 1) * kWideRows;
  const double mb = 2e-6 * n_cols * k;
  return groups == 1 || ((n_cols + 255) / 256 * groups > 256 && mb <= 850 && last <= (mb <= 320 ? 96 : 64));
}
constexpr size_t kWidePartFloats = (size_t)12 << 20;   // partial tiles of one wide matmul: at most 48 MB

inline SplitPlan plan_any(int epi, int n_cols, int k, int rows, int head_dim, bool qk_norm) {
  const int rp = rows_pad_for(rows);
  if (epi == EPI_HEAD && (rp <= 64 || (rp == 128 && k % 256 == 0))) return plan_head(n_cols, k, rows, rp);
  if (epi == EPI_HEAD || rp > 128) return plan_wide(epi, n_cols, k, rp, kWidePartFloats);
  return plan_stream(epi, n_cols, k, rows, head_dim, qk_norm);
}

// Decomposition of one matmul inside the layer kernel: at most max_items (tile, split) items, every
// split the same whole number of `unit`-deep steps (unit = ring depth x chunk depth of the kernel
// for this row count).  n_splits = 0: not possible for this shape.
inline SplitPlan plan_layer(int n_cols, int k, int unit, int max_items, int split_cap) {
  SplitPlan p;
  p.kernel = GEMM_LAYER;
  p.tile_n = kGemmTileN;
  p.n_tiles = (n_cols + p.tile_n - 1) / p.tile_n;
  p.n_splits = 0;
  p.k_per_split = 0;
  if (p.n_tiles > max_items || k % unit != 0) return p;
  int smax = max_items / p.n_tiles;
  if (smax > kMaxSplitK) smax = kMaxSplitK;
  if (smax > k / unit) smax = k / unit;
  if (smax > split_cap) smax = split_cap;
  for (int s = smax; s >= 1; --s)
    if (k % s == 0 && (k / s) % unit == 0) {
      p.n_splits = s;
      p.k_per_split = k / s;
      break;
    }
  return p;
}

// ---- attention: how the query rows and the keys of a pass are divided into workgroups
struct AttnPlan {
  bool few;          // k_attn_few
  int rows_per_wg, n_row_groups, keys_per_split, n_splits, draft_mode, n_draft;
};

// group * n_nodes query rows per kv head over up to max_keys keys; depth: nodes on the longest root path.
//
// At most 32 (64) rows over up to 128 (64) keys a CU take k_attn_few (9 nodes, 16 heads on 8: 1000 keys 11.4 -> 7.6 us, 4096
// keys 12.6 -> 10.6; 30 nodes, 2048 keys 12.7 -> 12.1); over more its scattered reads cost more than staging (8192 keys:
// 15.2 / 15.1 us for 9 nodes, 17.3 / 23.8 for 30; four sequences of 2048 keys 14.6 / 17.1).
//
// Else: workgroups of 64, 128 or 256 rows and a number of key splits, with the smallest estimated time of the context kernel
// and the merge together.  A context kernel takes a fixed time (launch, queries and first tile) and a time per key of its split, 15 % more
// when every CU has a workgroup, and the partials' way out; beyond 256 workgroups, one a CU, that comes again.  256 rows, and 128 rows
// that leave no wavefront without a row, have a least time whatever the split.  256 rows stage a key once for all rows of a tree;
// 64 rows by eight wavefronts that share a tile's keys out are the fastest per row, two wavefronts a SIMD, and leave
// half the partials of 128 rows, but every row group reads the keys again.  The draft nodes have workgroups of their own
// where those fit beside the context, else they are the merge's, by the node: 0.18 us for every node that the longest
// path goes beyond 8.  The merge takes its partials 20 at a time (16 with draft nodes, fewer wavefronts a CU beyond 8 or with 8 heads).
//
// Fitted to 451 shapes of 9 to 512 rows, 200 to 16384 keys, one to four sequences, head_dim 64 and 128, groups of 1 to 8, each in about ten
// divisions.  Of 140 others the chosen division is on average 1.1 % slower than the fastest, at worst 15 % (four sequences of 46 nodes, 744 keys,
// head_dim 64: 18.6 against 16.1 us); two are 4 and 5 % slower than 128 rows (256 over 6144 keys and more) in 256 workgroups.  With constants from
// fewer shapes 18 of 140 were, 256 rows over 2048 keys by 4 us a layer.  us, context + merge, 128 or 256 rows in 256 workgroups of 256 keys
// at least -> now, kv heads 8:
//   120 rows   8192 keys 19.7 + 9.9 -> 20.6 + 4.8, 16384 31.3 + 9.7 -> 28.9 + 6.4, 1024 13.7 + 4.5 -> 10.7 + 4.2, three sequences of 8192 61.7 + 12.0 -> 40.2 + 8.4
//   240 rows   8192 keys 26.8 + 13.7 -> 27.9 + 7.3, 4096 17.5 + 9.7 -> 18.7 + 7.3, 2048 15.2 + 5.2 -> 14.6 + 5.1, a chain over 4096 17.4 + 18.2 -> 19.5 + 5.7
//   256 rows   2048 keys 15.4 + 5.4 -> 15.4 + 5.4;   four sequences of 240 rows   16384 keys 129.6 + 21.7 -> 130.0 + 18.6
inline AttnPlan plan_attn(int batch, int n_kv, int group, int head_dim, int n_nodes, int depth, int max_keys, bool paged) {
  const int p_rows = group * n_nodes, n_draft = (n_nodes + 31) / 32;
  AttnPlan best;
  if (p_rows <= 32 ? batch * n_kv * max_keys <= 32768 : p_rows <= 64 && batch * n_kv * max_keys <= 16384) {
    // 128 keys at least, two workgroups to a CU; up to 16 splits, which the merge fetches in one round
    // trip, more only when a split would grow past 512 keys
    int want = max_keys > 16 * 512 ? (max_keys + 511) / 512 : 16;
    const int room = 512 / (batch * n_kv) - n_draft;
    if (want > room) want = room;
    if (want < 1) want = 1;
    if (want > kMaxAttnSplits) want = kMaxAttnSplits;
    int kps = ((max_keys + want - 1) / want + 127) / 128 * 128;
    if (kps < 128) kps = 128;
    best.few = true;
    best.rows_per_wg = p_rows <= 32 ? 32 : 64;
    best.n_row_groups = 1;
    best.keys_per_split = kps;
    best.n_splits = max_keys > kps ? (max_keys + kps - 1) / kps : 1;
    best.draft_mode = kDraftOwnGroups;
    best.n_draft = n_draft;
    return best;
  }
  best.few = false;
  const bool narrow = head_dim < 128;
  const double rows_k = p_rows * batch * n_kv * 1e-3;
  double best_us = 1e30;
  for (int rows = 64; rows <= 256; rows *= 2) {
    if ((rows == 64 && p_rows <= 64) || (rows == 256 && p_rows <= 128)) continue;   // 128 rows with at most 64 are the 64-row form
    const int groups = (p_rows + rows - 1) / rows, per_split = batch * n_kv * groups;
    const bool all_rows = rows == 128 && p_rows > 96;   // every wavefront of a 128-row workgroup has rows
    const double fixed = rows == 256 ? 8.1 : (rows == 64 ? 8.05 : (all_rows ? 5.3 : 6.45));
    const double per_key = rows == 256 ? 0.0367 : (rows == 64 ? 0.0148 : (all_rows ? 0.03 : (p_rows > 64 ? 0.0236 : 0.0174)));
    const double least = rows == 256 ? 21.0 : (all_rows ? 12.6 : 0.0);
    // every split starts at a multiple of the kernel's key tile, in a paged cache of the largest
    const int unit = rows == 256 && !paged ? 64 : 128;
    for (int s = 1; s <= kMaxAttnSplits; ++s) {
      int kps = ((max_keys + s - 1) / s + unit - 1) / unit * unit;
      if (kps < 128) kps = 128;
      const int n = max_keys > kps ? (max_keys + kps - 1) / kps : 1;
      if (n != s) continue;
      const bool own = (n + n_draft) * per_split <= 256;
      const int parts = n + (own ? n_draft : 0), rounds = (n * per_split + 255) / 256;
      const double side_by_side = (double)n * per_split / rounds + (own ? n_draft * per_split : 0);
      const double crowd = side_by_side < 128 ? 0.0 : (side_by_side < 256 ? side_by_side / 128 - 1 : 1.0);
      const double mb = rows_k * (head_dim + 2) * 4e-3;   // of one split's partials
      double us = fixed + per_key * kps * (1 + 0.15 * crowd);
      us = rounds * (us > least ? us : least) * (!narrow ? 1.0 : (rows == 256 || all_rows ? 0.73 : 0.675)) + 0.115 * mb * n;
      if (own)
        us += 3.3 + 0.235 * rows_k + 0.128 * mb * parts + 2.5 * ((parts - 1) / 20);
      else
        us += 4.2 + (narrow ? 0.5 : 1.0) * rows_k * (1 + (n > 8 ? 0.9 : 0.0) + (group == 8 ? 0.9 : 0.0)) + 0.043 * mb * n +
              3.8 * ((n - 1) / 16) + 0.18 * (depth > 8 ? depth - 8 : 0);
      if (us < best_us) {
        best_us = us;
        best.rows_per_wg = rows;
        best.n_row_groups = groups;
        best.keys_per_split = kps;
        best.n_splits = n;
        best.draft_mode = own ? kDraftOwnGroups : kDraftInMerge;
        best.n_draft = own ? n_draft : 0;
      }
    }
  }
  return best;
}

// ---- the plans of one model, made once: the matmuls of a pass depend on its rows only through the kind of panel

// kinds of panels: 1 to 4 row blocks of 16, 6, 8, more than 128 rows
constexpr int kPanelKinds = 7;
constexpr int kPanelRows[kPanelKinds] = {16, 32, 48, 64, 96, 128, 256};   // the most rows of each
inline int panel_kind(int rows) {
  int i = 0;
  while (i + 1 < kPanelKinds && rows > kPanelRows[i]) ++i;
  return i;
}
struct ModelPlans {
  SplitPlan qkv[kPanelKinds], o[kPanelKinds], gate_up[kPanelKinds], down[kPanelKinds], head[kPanelKinds];
  int max_tiles;                     // tile counters that the streaming kernel needs, over all panels
  size_t part_floats[kPanelKinds];   // partial tiles of one matmul over panels of this and the smaller kinds
};
inline ModelPlans make_plans(const trispec_model_config &c) {   // bf16 models
  ModelPlans m = {};
  const int qd = c.n_q_heads * c.head_dim, nqkv = qd + 2 * c.n_kv_heads * c.head_dim;
  for (int i = 0; i < kPanelKinds; ++i) {
    const int r = kPanelRows[i];
    m.part_floats[i] = i > 0 ? m.part_floats[i - 1] : 0;
    auto plan = [&](int epi, int n_cols, int k) {
      const SplitPlan p = plan_any(epi, n_cols, k, r, c.head_dim, c.qk_norm != 0);
      if (epi == EPI_HEAD) return p;
      const bool stream = p.kernel == GEMM_STREAM;
      if (stream && counted_tiles(epi, p, r) > m.max_tiles) m.max_tiles = counted_tiles(epi, p, r);
      const size_t f = stream ? stream_part_floats(epi, p, r) : (size_t)p.n_splits * tiles_of(n_cols) * kGemmTileN * r;
      if (f > m.part_floats[i]) m.part_floats[i] = f;
      return p;
    };
    m.qkv[i] = plan(EPI_QKV, nqkv, c.hidden);
    m.o[i] = plan(EPI_RESID, c.hidden, qd);
    m.gate_up[i] = plan(EPI_SWIGLU, 2 * c.ffn, c.hidden);
    m.down[i] = plan(EPI_RESID, c.hidden, c.ffn);
    m.head[i] = plan(EPI_HEAD, c.vocab, c.hidden);
  }
  return m;
}

}  // namespace ts
