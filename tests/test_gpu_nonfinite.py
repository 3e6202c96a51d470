"""Values that are not finite: a NaN that a row may see reaches its results whichever kernel adds the row up."""
import numpy as np
import pytest

from workloads import SHAPES, gen_draft_tokens, gen_kv_cache, gen_tree, tree_depths
from gpu_helpers import Case, device_model

pytestmark = pytest.mark.gpu

TB = SHAPES["tiny_bf16"].with_(n_layers=1, vocab=600)


def synthetic_case(shape, seed, ctx, parents):
    k, v = gen_kv_cache(shape, len(ctx), max(ctx), seed, 0)
    return Case(shape, seed, [k[b][None, :, :n].astype(np.float64) for b, n in enumerate(ctx)],
                [v[b][None, :, :n].astype(np.float64) for b, n in enumerate(ctx)],
                np.stack([gen_draft_tokens(p, shape.vocab - 1, seed + b) for b, p in enumerate(parents)]),
                np.stack(parents), np.stack([n + tree_depths(p) for n, p in zip(ctx, parents)]))


def star(n):
    return np.array([-1] + [0] * (n - 1), dtype=np.int32)


# ------------------------------------------------------------------ attention
# (query heads over 2 kv heads, contexts, tree, spoilt node): k_attn_few over 32 and 64 rows, workgroups of 128
# and 256 rows with blocks of draft nodes, draft nodes in the merge
DRAFTS = {
    "few64_root": (2, (300,), star(40), 0),
    "own128_root": (8, (300,), star(40), 0),
    "own128_inner": (4, (300,), gen_tree(100, 8, 4, 1), 47),
    "own256_inner": (4, (6200,), gen_tree(100, 8, 4, 1), 47),
    "in_merge_root": (4, (16380, 300, 0, 77), star(40), 0),
}


@pytest.mark.parametrize("paged", [False, True], ids=["dense", "paged"])
@pytest.mark.parametrize("name", list(DRAFTS))
def test_a_spoilt_node_reaches_every_descendant(name, paged):
    """The draft nodes are added up in blocks of 32.  A node with a NaN score that is a row's only ancestor in its
    block must not pass for a block without ancestors."""
    heads, ctx, parents, hit = DRAFTS[name]
    n = len(parents)
    below = np.zeros(n, dtype=bool)
    alone = []                                   # rows that see nothing else of the spoilt node's block
    for i in range(n):
        path, j = [], i
        while j >= 0:
            path.append(j)
            j = parents[j]
        below[i] = hit in path
        if below[i] and [j for j in path if j // 32 == hit // 32] == [hit]:
            alone.append(i)
    assert len(alone) > 2
    case = synthetic_case(TB.with_(n_q_heads=heads), 700 + len(name), ctx, [parents] * len(ctx))
    model = device_model(case.shape, case.seed)
    clean = case.run_gpu(0.0, model=model, paged=paged)["logits"].copy()
    bad = case.shape.vocab - 1                   # drafted nowhere else
    model.tensors["embed"][bad].fill_(float("inf"))
    case.tokens[:, hit] = bad
    got = case.run_gpu(0.0, model=model, paged=paged)["logits"]
    assert np.isfinite(clean).all()
    assert not np.isfinite(got[:, below]).any(axis=-1).any()
    # the rest: the same terms, in another order where a block holds a value that is not finite: the bar of
    # logits in test_gpu_parity.py
    if not below.all():
        assert np.abs(got[:, ~below] - clean[:, ~below]).max() <= 2e-3


# (query heads, nodes, contexts, first keys that are NaN: whole splits of the context, none in part)
CONTEXTS = {
    "few32": (4, 9, (600,), 128),
    "few64": (4, 25, (600,), 128),
    "own128": (4, 100, (600,), 256),
    "own256": (4, 100, (6200,), 256),
    "in_merge": (4, 40, (16380, 600, 700, 513), 512),
}


@pytest.mark.parametrize("paged", [False, True], ids=["dense", "paged"])
@pytest.mark.parametrize("name", list(CONTEXTS))
def test_a_stretch_of_spoilt_context_is_not_skipped(name, paged):
    """Keys that are all NaN over exactly one split of the context must not pass for a split without keys."""
    heads, nodes, ctx, spoilt = CONTEXTS[name]
    case = synthetic_case(TB.with_(n_q_heads=heads), 800 + len(name), ctx, [gen_tree(nodes, 8, 4, 3)] * len(ctx))
    for k in case.k_ctx:
        k[:, :, :spoilt] = np.nan
    got = case.run_gpu(0.0, paged=paged)["logits"]
    assert not np.isfinite(got).any()
