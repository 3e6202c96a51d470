"""Every division of attention into workgroups (64, 128 and 256 rows, key groups, draft nodes in workgroups of their own or in the
merge), at ragged row groups and splits, against the oracle.  tests/test_attn_plans.py asks the planner which form each case takes."""
import numpy as np
import pytest

from workloads import SHAPES, gen_draft_tokens, gen_kv_cache, gen_tree, tree_depths
from gpu_helpers import Case, compare_decisions

TB = SHAPES["tiny_bf16"].with_(n_layers=1, vocab=600)
W8 = TB.with_(n_q_heads=16, n_kv_heads=8)                 # 2 query heads to each of 8 kv heads
W16 = TB.with_(n_q_heads=32, n_kv_heads=16)
G4 = TB.with_(n_q_heads=8, n_kv_heads=2)
D64 = TB.with_(n_q_heads=24, n_kv_heads=8, head_dim=64)   # groups of 3
# (model, sequences, nodes, contexts, tree or chain), named for who evaluates the draft nodes and the rows of a workgroup
FORMS = {
    "own64_rows120": (W8, 1, 60, (8100,), "tree"),
    "merge64_three_sequences": (W8, 3, 51, (4100, 77, 0), "tree"),
    "own64_rows102": (W8, 1, 51, (1030,), "tree"),
    "own128_three_sequences": (W8, 3, 60, (2050, 20, 700), "tree"),
    "own128_rows120_chain": (W8, 1, 60, (4001,), "chain"),
    "merge128_rows120": (W16, 3, 60, (2050, 700, 131), "tree"),
    "own64_rows74_chain": (W8, 1, 37, (3001,), "chain"),
    "merge128_rows80": (W16, 4, 40, (4100, 3, 640, 1499), "tree"),
    "own256_rows240": (W16.with_(n_q_heads=64), 2, 60, (2050, 1000), "tree"),
    "own128_rows240_chain": (W8.with_(n_q_heads=32), 1, 60, (2050,), "chain"),
    "own256_rows512_chain": (G4, 2, 128, (9001, 300), "chain"),
    "merge256_d64_rows160": (W16.with_(n_q_heads=64, head_dim=64), 3, 40, (2050, 128, 0), "tree"),
    "own128_d64_rows69": (D64, 1, 23, (6001,), "tree"),
    "own64_d64_rows180": (D64, 1, 60, (5003,), "tree"),
    "own64_rows200": (G4, 1, 50, (8190,), "tree"),
}


def parents_of(kind, nodes, seed):
    return np.arange(-1, nodes - 1, dtype=np.int32) if kind == "chain" else gen_tree(nodes, 8, 4, 600 + seed)


@pytest.mark.gpu
@pytest.mark.parametrize("paged", [False, True], ids=["dense", "paged"])
@pytest.mark.parametrize("name", list(FORMS))
def test_forms(name, paged):
    shape, batch, nodes, ctx, kind = FORMS[name]
    parents = [parents_of(kind, nodes, b) for b in range(batch)]
    k, v = gen_kv_cache(shape, batch, max(ctx), 41, 0)
    case = Case(shape, 41, [k[b][None, :, :n].astype(np.float64) for b, n in enumerate(ctx)],
                [v[b][None, :, :n].astype(np.float64) for b, n in enumerate(ctx)],
                np.stack([gen_draft_tokens(p, shape.vocab, 41 + b) for b, p in enumerate(parents)]), np.stack(parents),
                np.stack([n + tree_depths(p) for n, p in zip(ctx, parents)]))
    got, want = case.run_gpu(0.5, paged=paged), case.run_oracle()
    for b in range(batch):   # the bar of logits of every bf16 test of one or two layers
        assert np.abs(got["logits"][b] - want[b]["logits"]).max() <= 2e-3
    compare_decisions(case, got, want, 0.5, 0)
