// Reads lines "batch n_kv group head_dim nodes depth keys paged" and prints the division of attention that the library makes for
// each: "few rows_per_workgroup row_groups keys_per_split splits draft_mode draft_blocks".
#include <cstdio>

#include "plan.hpp"

int main() {
  int b, kv, g, d, n, depth, keys, paged;
  while (scanf("%d %d %d %d %d %d %d %d", &b, &kv, &g, &d, &n, &depth, &keys, &paged) == 8) {
    const ts::AttnPlan p = ts::plan_attn(b, kv, g, d, n, depth, keys, paged != 0);
    printf("%d %d %d %d %d %d %d\n", (int)p.few, p.rows_per_wg, p.n_row_groups, p.keys_per_split, p.n_splits, p.draft_mode, p.n_draft);
  }
  return 0;
}
