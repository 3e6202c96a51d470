"""The k splits of a tile meet: every workgroup of the tile finishes row blocks of it, or the last to arrive finishes
those of workgroups that have left.  With a wait of one tick (10 ns) many leave, as the words that they met at show; the sums
are added in the same order, so that a pass leaves the same bits either way."""
import numpy as np
import pytest
import torch

from paper_2601_23180_amd import binding
from workloads import SHAPES, gen_tree
from test_gpu_parity import full_check, make_case

pytestmark = pytest.mark.gpu

# batch, nodes, hidden, query heads, kv heads, head_dim, ffn, qk_norm: 3, 4, 6 and 8 row blocks, the last one ragged or without
# any row; as many splits as blocks and more; q and k with norms of their own (two groups of 64 rows over more than 64).
# test_plans.py asks the planner which products meet.
SIZES = [(1, 33, 1024, 8, 4, 128, 1536, 0), (1, 48, 512, 4, 2, 64, 4096, 1), (1, 60, 2048, 16, 8, 128, 6144, 0),
         (4, 16, 4096, 8, 8, 128, 4096, 0), (1, 65, 1792, 3, 3, 128, 1024, 0), (3, 27, 1472, 12, 4, 64, 4032, 0),
         (3, 37, 2048, 16, 8, 128, 6144, 1), (2, 64, 1024, 8, 8, 128, 3072, 0), (2, 23, 1536, 6, 6, 64, 1024, 0),
         (5, 21, 2688, 4, 4, 64, 1024, 0)]


@pytest.mark.parametrize("size", SIZES, ids=["rows%d_%d" % (s[0] * s[1], s[2]) for s in SIZES])
def test_splits_that_leave(size):
    batch, nodes, hidden, nq, nkv, d, ffn, norm = size
    shape = SHAPES["tiny_bf16"].with_(n_layers=3, hidden=hidden, n_q_heads=nq, n_kv_heads=nkv, head_dim=d, ffn=ffn,
                                      qk_norm=bool(norm), vocab=300, lm_head_std=3 / hidden ** 0.5)
    seed = 900 + hidden + nodes
    case = make_case(shape, seed, [20 + 17 * b for b in range(batch)], [gen_tree(nodes, 9, 4, seed + b) for b in range(batch)])
    stay, _, _ = full_check(case, thresholds=(0.5,))
    ver, kv, pos = stay["_ver"], stay["_kv"], torch.from_numpy(case.positions).cuda()

    def again():
        """One more pass over the same cache slots: logits, and the workspace as it leaves it."""
        out = ver.verify(kv, stay["_tok"], case.parents, pos, 0.5)
        torch.cuda.synchronize()
        assert out["status"].item() == 0
        return ver.logits.cpu().numpy(), ver.workspace.view(torch.int32).cpu().numpy()
    before = again()
    lib = binding.lib()
    try:
        lib.trispec_debug_set_spin_limit(1)
        leave = again()
    finally:
        lib.trispec_debug_set_spin_limit(0)
    after = again()
    for logits, _ in (before, leave, after):
        assert np.array_equal(stay["logits"], logits)
    # nothing in the workspace tells the passes apart but the words of the last launch that met there: as many arrivals (bits
    # 0 - 7), and a bit for each workgroup that has left
    changed = before[1] != leave[1]
    assert np.array_equal(before[1][changed] & 255, leave[1][changed] & 255)
    departures = [sum(bin(w >> 8).count("1") for w in words[changed].tolist()) for words in (before[1], leave[1])]
    assert departures[1] > departures[0]
