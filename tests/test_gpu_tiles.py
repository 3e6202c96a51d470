"""Edges of the matmul kernels' tiles and splits, whole passes of one-layer models against the oracle:
row counts at both ends of every panel size, reductions of 1, 2, 3 and more 64-deep blocks per split
(every tail of the software pipelines), output widths that end inside a tile.  Bars: those of
test_gpu_parity.py (logits 2e-3 absolute, decisions exact outside flagged ties)."""
import numpy as np
import pytest
import torch

from workloads import SHAPES, gen_tree
from oracle import adapter
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
    # larger products: QKV in 96 columns, gate + up in 48 and 112, runs that are no whole number of rounds
    ("rows60_qkv96_gate_up48", 1, 60, TB.with_(hidden=4096, ffn=6144, n_q_heads=32, n_kv_heads=8, lm_head_std=0.1)),
    ("rows16_gate_up112_odd_head64", 1, 16, TB.with_(hidden=448, ffn=14336, head_dim=64, n_q_heads=7, n_kv_heads=7,
                                                     lm_head_std=0.3)),
    ("rows48_gate_up112_ragged", 3, 16, TB.with_(hidden=576, ffn=12352, n_q_heads=4, lm_head_std=0.3)),
    ("rows17_wide_down", 1, 17, TB.with_(hidden=4096, ffn=4096, n_q_heads=2, lm_head_std=0.1)),
    # LM head: more tiles than places over at most 32 rows (two passes of two or three sub-tiles, a ragged last one)
    ("rows9_vocab_passes", 1, 9, TB.with_(hidden=512, ffn=256, vocab=70001, lm_head_std=0.3)),
    ("rows32_vocab_passes", 4, 8, TB.with_(hidden=512, ffn=256, vocab=132000, lm_head_std=0.3)),
    # more than 64 rows
    ("rows100_gate_up96", 1, 100, TB.with_(hidden=512, ffn=12288, lm_head_std=0.3)),
    ("rows111_whole_heads", 3, 37, TB.with_(hidden=1024, ffn=6144, n_q_heads=16, n_kv_heads=8, qk_norm=True, lm_head_std=0.2)),
    ("rows65_one_block", 1, 65, TB.with_(hidden=64, ffn=64, head_dim=64, n_q_heads=1, n_kv_heads=1, lm_head_std=0.8)),
    ("rows96_two_blocks", 3, 32, TB.with_(hidden=128, ffn=128, lm_head_std=0.6)),
    ("rows128_three_blocks_ragged", 2, 64, TB.with_(hidden=192, ffn=320, head_dim=64, n_q_heads=6, n_kv_heads=3,
                                                    vocab=777, lm_head_std=0.5)),
    ("rows129_five_blocks", 3, 43, TB.with_(hidden=320, ffn=192, vocab=513, lm_head_std=0.4)),
    ("rows256_splits", 4, 64, TB.with_(hidden=1024, ffn=1472, n_q_heads=8, vocab=1024, lm_head_std=0.2)),
    ("rows250_many_splits_qk_norm", 5, 50, TB.with_(hidden=256, ffn=4096, qk_norm=True, lm_head_std=0.4)),
    ("rows129_odd_chunks", 3, 43, TB.with_(hidden=320, ffn=448, lm_head_std=0.4)),
    # LM head in more than one round of workgroups: row groups one after the other (a last one of 1 and of 96 rows), and side by side
    ("rows129_vocab_apart", 3, 43, TB.with_(hidden=192, ffn=64, vocab=33001, lm_head_std=0.5)),
    ("rows224_vocab_apart", 4, 56, TB.with_(hidden=64, ffn=64, vocab=32769, lm_head_std=0.8)),
    ("rows225_vocab_side_by_side", 5, 45, TB.with_(hidden=64, ffn=64, vocab=33001, lm_head_std=0.8)),
]


# The streaming kernel in every tile width that a model of at most 30M weights a layer takes, over every number of row blocks,
# in one k split and in several (test_plans.py looks the plans up): batch, nodes, hidden, query heads, kv heads,
# head_dim, ffn, qk_norm
WIDTHS = [
    (1, 1, 64, 32, 4, 128, 8448, 0), (2, 4, 64, 10, 2, 64, 64, 1), (1, 8, 1536, 8, 1, 128, 64, 1),
    (3, 3, 4160, 1, 1, 64, 64, 1), (1, 11, 16512, 1, 1, 64, 64, 1), (2, 6, 2816, 14, 2, 128, 128, 0),
    (2, 7, 64, 8, 1, 64, 12352, 0), (5, 3, 64, 2, 1, 64, 6400, 0), (2, 8, 64, 2, 1, 128, 4224, 1),
    (4, 4, 8576, 1, 1, 64, 64, 0), (1, 19, 64, 32, 4, 128, 18624, 0), (5, 4, 4160, 1, 1, 64, 64, 0),
    (3, 8, 1472, 12, 2, 128, 64, 1), (1, 25, 64, 2, 1, 128, 6848, 1), (1, 26, 2624, 3, 3, 128, 64, 0),
    (2, 14, 64, 1, 1, 64, 4224, 1), (7, 4, 16512, 1, 1, 64, 64, 0), (1, 29, 8320, 1, 1, 64, 64, 1),
    (1, 29, 2816, 20, 4, 128, 192, 1), (4, 8, 64, 3, 1, 64, 12416, 0), (1, 33, 64, 2, 1, 64, 8448, 1),
    (5, 7, 64, 4, 2, 64, 4160, 0), (2, 19, 64, 2, 2, 128, 6272, 1), (8, 5, 2816, 20, 4, 128, 128, 0),
    (1, 41, 4160, 1, 1, 64, 64, 0), (1, 43, 2112, 8, 1, 128, 64, 1), (2, 23, 8384, 1, 1, 64, 64, 1),
    (1, 46, 16448, 1, 1, 64, 64, 1), (3, 16, 64, 28, 4, 128, 13632, 0), (5, 10, 16832, 1, 1, 64, 64, 1),
    (1, 51, 64, 1, 1, 128, 6272, 1), (3, 17, 8320, 1, 1, 64, 64, 0), (1, 53, 64, 1, 1, 64, 12352, 1),
    (5, 11, 64, 1, 1, 128, 4160, 0), (3, 19, 2304, 7, 1, 128, 64, 1), (3, 19, 2816, 24, 4, 128, 64, 0),
    (1, 59, 4160, 1, 1, 64, 64, 1), (4, 16, 64, 28, 4, 128, 8384, 0), (6, 11, 2304, 6, 1, 128, 64, 1),
    (3, 23, 64, 3, 1, 64, 4224, 1), (2, 37, 2752, 24, 3, 128, 64, 0), (3, 25, 8448, 1, 1, 64, 64, 0),
    (2, 42, 64, 5, 1, 64, 64, 0), (7, 13, 64, 1, 1, 128, 6784, 1), (7, 13, 128, 28, 4, 128, 8768, 0),
    (3, 32, 4160, 1, 1, 64, 64, 1), (3, 33, 64, 32, 4, 128, 6720, 0), (2, 53, 2752, 24, 4, 128, 64, 1),
    (6, 18, 8320, 1, 1, 64, 64, 1), (2, 55, 64, 5, 1, 64, 64, 1), (1, 123, 4160, 1, 1, 64, 64, 0),
    (4, 31, 2688, 7, 1, 128, 64, 0), (1, 125, 64, 1, 1, 64, 18496, 0), (4, 32, 64, 5, 1, 64, 4160, 0),
    # three row blocks and more: the k splits of a tile finished by one workgroup, and by all of them
    (5, 12, 384, 1, 1, 64, 64, 0), (2, 31, 576, 1, 1, 64, 64, 1), (1, 83, 576, 1, 1, 64, 64, 1),
    (1, 41, 640, 1, 1, 64, 64, 1), (4, 26, 704, 1, 1, 64, 64, 1), (3, 13, 640, 1, 1, 128, 64, 1),
    (1, 108, 3584, 1, 1, 64, 64, 1), (1, 48, 64, 105, 15, 128, 64, 0), (1, 49, 64, 105, 15, 128, 64, 0),
    (2, 23, 1536, 6, 6, 64, 64, 0), (5, 11, 1280, 8, 8, 64, 64, 0), (1, 73, 1792, 3, 3, 128, 64, 0),
    (5, 21, 2688, 4, 4, 64, 64, 0), (2, 39, 640, 48, 6, 64, 64, 0), (3, 12, 2816, 21, 3, 64, 64, 0),
    (1, 60, 4288, 21, 3, 64, 64, 1), (1, 43, 2688, 15, 15, 128, 64, 0), (1, 51, 1472, 45, 15, 128, 64, 0),
    (1, 45, 1600, 45, 15, 128, 64, 0),
]
CASES += [("widths_rows%d_%d" % (w[0] * w[1], i), w[0], w[1],
           TB.with_(hidden=w[2], n_q_heads=w[3], n_kv_heads=w[4], head_dim=w[5], ffn=w[6], qk_norm=bool(w[7]), vocab=200,
                    lm_head_std=3 / w[2] ** 0.5)) for i, w in enumerate(WIDTHS)]


@pytest.mark.parametrize("name,batch,nodes,shape", CASES, ids=[c[0] for c in CASES])
def test_tile_edges(name, batch, nodes, shape):
    seed = 300 + len(name)
    parents = [gen_tree(nodes, 9, 4, seed + b) if nodes > 1 else np.array([-1], dtype=np.int32) for b in range(batch)]
    full_check(make_case(shape, seed, [20 + 17 * b for b in range(batch)], parents), thresholds=(0.0, 0.5))


# The adapter's plain product: (batch, nodes, hidden, adapter width).  Up to 128 rows, the streaming kernel: one split,
# several, finished by one workgroup or by all of a tile, several that need more tile counters than the layers do (one
# split instead); more rows: one split in 128- and
# in 256-column tiles, k splits finished by the second launch; widths that end inside a tile.
ADAPTERS = {
    "rows23_splits": (1, 23, 1472, 132),
    "rows64_no_counters": (1, 64, 1024, 2052),
    "rows100_one_split": (1, 100, 256, 200),
    "rows100_splits_ragged_k": (1, 100, 1472, 132),
    "rows34_one_split": (1, 34, 64, 132),
    "rows37_splits": (1, 37, 576, 132),
    "rows37_meet": (1, 37, 832, 132),
    "rows57_one_split": (1, 57, 64, 200),
    "rows60_meet": (1, 60, 1024, 132),
    "rows75_one_split": (1, 75, 64, 200),
    "rows68_splits": (1, 68, 448, 132),
    "rows90_meet": (3, 30, 4928, 132),
    "rows124_meet": (2, 62, 2368, 132),
    "rows250_splits": (5, 50, 1024, 260),
    "rows130_one_split": (2, 65, 64, 200),
    "rows130_wide_tiles": (2, 65, 64, 16500),
}


@pytest.mark.parametrize("name", list(ADAPTERS))
def test_adapter_edges(name):
    batch, nodes, hidden, dim = ADAPTERS[name]
    shape, seed = TB.with_(hidden=hidden, ffn=256, vocab=300, lm_head_std=0.2), 600 + len(name)
    case = make_case(shape, seed, [20 + 3 * b for b in range(batch)], [gen_tree(nodes, 9, 4, seed + b) for b in range(batch)])
    want = case.run_oracle()
    gpu = case.run_gpu(0.5)
    rng = np.random.default_rng(seed)
    w = torch.from_numpy((rng.standard_normal((dim, hidden)) * 0.05).astype(np.float32)).cuda().to(torch.bfloat16)
    bias = rng.standard_normal(dim).astype(np.float32)
    ver = gpu["_ver"]
    out = ver.set_adapter(w, torch.from_numpy(bias).cuda())
    out.fill_(float("nan"))
    ver.verify(gpu["_kv"], gpu["_tok"], case.parents, torch.from_numpy(case.positions).cuda(), 0.5)
    torch.cuda.synchronize()
    y = out.cpu().numpy().reshape(batch, nodes, dim)
    for b in range(batch):
        ref = adapter(want[b]["final_hidden"], w.float().cpu().numpy(), bias)
        err = np.abs(y[b] - ref).max(axis=1) / np.abs(ref).max(axis=1)
        assert err.max() <= 3e-4, (b, err.max())     # bf16 hi + lo operands, as test_feature_layers_and_adapter


# Who evaluates the draft nodes of an attention call, and with how many rows a workgroup (test_attn_plans.py asks the planner):
# (batch, nodes, query heads, kv heads, contexts)
ATTN_CASES = {
    "rows18_own_workgroups": (1, 9, 4, 2, (300,)),
    "rows64_page_ends": (2, 32, 4, 2, (256, 257)),
    "rows58_batch": (3, 29, 4, 2, (0, 31, 1500)),
    "rows4_one_node_long": (1, 1, 8, 2, (9000,)),
    "rows200_own_workgroups": (1, 100, 4, 2, (300,)),
    "rows512_chain_blocks": (1, 128, 8, 2, (65,)),
    "rows128_unequal": (8, 32, 8, 2, (13000, 300, 64, 0, 77, 12999, 500, 9)),
    # few rows over many keys: the wavefronts share the keys of a tile out (four, four of eight, two of eight)
    "rows18_shared_keys": (2, 9, 4, 2, (16500, 300)),
    "rows52_shared_keys": (2, 26, 4, 2, (9000, 8001)),
    "rows74_shared_keys": (2, 37, 16, 8, (2050, 130)),
    # 4 splits for each of 64 (sequence, kv head) fill the chip: the draft nodes stay with the merge
    "rows80_in_merge": (4, 40, 32, 16, (1000, 128, 0, 500)),
}


def attn_case(name):
    from gpu_helpers import Case
    from workloads import gen_draft_tokens, gen_kv_cache, tree_depths
    batch, nodes, heads, kv_heads, ctx = ATTN_CASES[name]
    shape, seed = TB.with_(n_q_heads=heads, n_kv_heads=kv_heads, vocab=600), 500 + len(name)
    if nodes == 128:
        parents = [np.arange(-1, nodes - 1, dtype=np.int32)]
    else:
        parents = [gen_tree(nodes, 8, 4, seed + b) if nodes > 1 else np.array([-1], dtype=np.int32) for b in range(batch)]
    k, v = gen_kv_cache(shape, batch, max(ctx), seed, 0)
    return Case(shape, seed, [k[b][None, :, :n].astype(np.float64) for b, n in enumerate(ctx)],
                [v[b][None, :, :n].astype(np.float64) for b, n in enumerate(ctx)],
                np.stack([gen_draft_tokens(p, shape.vocab, seed + b) for b, p in enumerate(parents)]),
                np.stack(parents), np.stack([n + tree_depths(p) for n, p in zip(ctx, parents)]))


@pytest.mark.parametrize("paged", [False, True], ids=["dense", "paged"])
@pytest.mark.parametrize("name", list(ATTN_CASES))
def test_attention_forms(name, paged):
    full_check(attn_case(name), thresholds=(0.0, 0.5), paged=paged)


@pytest.mark.parametrize("name", ["rows18_own_workgroups", "rows58_batch", "rows200_own_workgroups",
                                  "rows128_unequal", "rows80_in_merge"])
def test_infinite_values_stay_on_their_branch(name):
    """A draft token whose embedding is not finite spoils its own subtree and nothing else.  Blocks of draft
    nodes with such a value are added up node by node instead of by matrix instructions: at most 128 fp32
    terms in another order, 128 * 2^-24 of an attention output of order 1, which the 16-bit high + low
    operands of the matmuls after it (2^-17 each) in this one layer carry into logits of up to about 10: the
    2e-3 of the other cases covers it.  (test_gpu_nonfinite.py has the nodes that are a row's only ancestor in
    their block.)"""
    from gpu_helpers import device_model
    case = attn_case(name)
    model = device_model(case.shape, case.seed)
    bad = case.shape.vocab - 1
    case.tokens[case.tokens == bad] = 0
    clean = case.run_gpu(0.0, model=model)["logits"].copy()
    model.tensors["embed"][bad].fill_(float("inf"))
    spoilt = np.zeros((case.batch, case.n_nodes), dtype=bool)
    for b in range(case.batch):
        hit = case.n_nodes // 2
        case.tokens[b][hit] = bad
        for i in range(case.n_nodes):
            spoilt[b, i] = i == hit or (case.parents[b][i] >= 0 and spoilt[b, case.parents[b][i]])
    got = case.run_gpu(0.0, model=model)["logits"]
    assert np.isfinite(clean).all() and not np.isfinite(got[spoilt]).all(axis=-1).any()
    assert np.abs(got[~spoilt] - clean[~spoilt]).max() <= 2e-3
