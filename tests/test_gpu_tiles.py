"""Edges of the matmul kernels' tiles and splits, whole passes of one-layer models against the oracle:
row counts at both ends of every panel size, reductions of 1, 2, 3 and more 64-deep blocks per split
(every tail of the software pipelines), output widths that end inside a tile.  Bars: those of
test_gpu_parity.py (logits 2e-3 absolute, decisions exact outside flagged ties)."""
import numpy as np
import pytest

from workloads import SHAPES, gen_tree
from test_gpu_parity import full_check, make_case

pytestmark = pytest.mark.gpu

TB = SHAPES["tiny_bf16"].with_(n_layers=1, vocab=1000)
CASES = [
    # (batch, nodes, shape): up to 64 rows; fewer 64-deep blocks than wavefronts, k that is no whole number of
    # chunks, heads of 64 and 128 with and without their own norm, tiles that end past the last column
    ("row1_one_block", 1, 1, TB.with_(hidden=64, ffn=64, head_dim=64, n_q_heads=1, n_kv_heads=1, lm_head_std=0.8)),
    ("rows23_ragged_k", 1, 23, TB.with_(hidden=192, ffn=320, n_q_heads=3, n_kv_heads=3, vocab=777, lm_head_std=0.5)),
    ("rows32_ragged_k_qk_norm", 2, 16, TB.with_(hidden=320, ffn=448, n_q_heads=3, n_kv_heads=1, qk_norm=True,
                                                lm_head_std=0.4)),
    ("rows33_head64_qk_norm", 3, 11, TB.with_(hidden=832, ffn=1088, head_dim=64, n_q_heads=6, n_kv_heads=2,
                                              qk_norm=True, vocab=513, lm_head_std=0.3)),
    ("rows46_half_heads_many_splits", 2, 23, TB.with_(hidden=1472, ffn=4032, n_q_heads=8, lm_head_std=0.2)),
    ("rows64_whole_heads", 1, 64, TB.with_(hidden=1344, ffn=1024, n_q_heads=8, qk_norm=True, vocab=129,
                                           lm_head_std=0.2)),
    ("rows64_chunks", 4, 16, TB.with_(hidden=2048, ffn=2560, n_q_heads=16, n_kv_heads=8, lm_head_std=0.15)),
    # more than 64 rows
    ("rows65_one_block", 1, 65, TB.with_(hidden=64, ffn=64, head_dim=64, n_q_heads=1, n_kv_heads=1, lm_head_std=0.8)),
    ("rows96_two_blocks", 3, 32, TB.with_(hidden=128, ffn=128, lm_head_std=0.6)),
    ("rows128_three_blocks_ragged", 2, 64, TB.with_(hidden=192, ffn=320, head_dim=64, n_q_heads=6, n_kv_heads=3,
                                                    vocab=777, lm_head_std=0.5)),
    ("rows129_five_blocks", 3, 43, TB.with_(hidden=320, ffn=192, vocab=513, lm_head_std=0.4)),
    ("rows256_splits", 4, 64, TB.with_(hidden=1024, ffn=1472, n_q_heads=8, vocab=1024, lm_head_std=0.2)),
    ("rows250_many_splits_qk_norm", 5, 50, TB.with_(hidden=256, ffn=4096, qk_norm=True, lm_head_std=0.4)),
]


@pytest.mark.parametrize("name,batch,nodes,shape", CASES, ids=[c[0] for c in CASES])
def test_tile_edges(name, batch, nodes, shape):
    seed = 300 + len(name)
    parents = [gen_tree(nodes, 9, 4, seed + b) if nodes > 1 else np.array([-1], dtype=np.int32) for b in range(batch)]
    full_check(make_case(shape, seed, [20 + 17 * b for b in range(batch)], parents), thresholds=(0.0, 0.5))
