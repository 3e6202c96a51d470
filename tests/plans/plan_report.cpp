// Reads lines "epilogue columns k rows head_dim qk_norm" and prints the plan that the library makes for each:
// "kernel width tiles splits counters floats-of-partial-tiles built meets apart" (the four before the last of the streaming kernel only; meets:
// all workgroups of a tile finish it; apart: the LM head's row groups in the wide kernel).
#include <cstdio>

#include "plan.hpp"

int main() {
  for (int tiles = 1; tiles <= 512; ++tiles)   // the wide kernel's item / tiles
    for (int item = 0; item < 16 * tiles; ++item)
      if (ts::wide_split(item, tiles, ts::wide_tiles_inv(tiles)) != item / tiles) return 1;
  int epi, n, k, rows, d, norm;
  while (scanf("%d %d %d %d %d %d", &epi, &n, &k, &rows, &d, &norm) == 6) {
    const ts::SplitPlan p = ts::plan_any(epi, n, k, rows, d, norm != 0);
    const bool stream = p.kernel == ts::GEMM_STREAM;
    const int rb = ts::row_groups(epi, p, rows) > 1 ? 4 : ts::row_blocks(rows);   // row blocks of a tile
    printf("%d %d %d %d %d %zu %d %d %d\n", p.kernel, p.tile_n, p.n_tiles, p.n_splits, ts::counted_tiles(epi, p, rows),
           stream ? ts::stream_part_floats(epi, p, rows) : (size_t)0, stream ? (int)ts::stream_built(epi, p.tile_n, rb) : 0,
           stream ? (int)ts::tile_meets(epi, rb, p.n_splits) : 0,
           p.kernel == ts::GEMM_WIDE && epi == ts::EPI_HEAD ? (int)ts::wide_apart(n, k, rows) : 0);
  }
  return 0;
}
