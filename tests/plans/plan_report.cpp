// Reads lines "epilogue columns k rows head_dim qk_norm" and prints the plan that the library makes for each:
// "streaming width tiles splits counters floats-of-partial-tiles" (the last two of the streaming kernel only).
#include <cstdio>

#include "plan.hpp"

int main() {
  int epi, n, k, rows, d, norm;
  while (scanf("%d %d %d %d %d %d", &epi, &n, &k, &rows, &d, &norm) == 6) {
    const ts::SplitPlan p = ts::plan_any(epi, n, k, rows, d, norm != 0);
    printf("%d %d %d %d %d %zu\n", p.stream, p.tile_n, p.n_tiles, p.n_splits, ts::counted_tiles(epi, p, rows),
           p.stream ? ts::stream_part_floats(epi, p, rows) : (size_t)0);
  }
  return 0;
}
