"""Values that are not finite, and logits near the end of the fp32 range: a NaN that a row may see reaches its
results whichever kernel adds the row up, no statistic makes a NaN of numbers or a number of a NaN, and a node
whose statistic is a NaN is never trusted."""
import numpy as np
import pytest
import torch

from oracle import CRIT_TOP1
from paper_2601_23180_amd import model_from_arrays
from workloads import SHAPES, WeightSource, gen_draft_tokens, gen_kv_cache, gen_tree, tree_depths
from workloads.gen import bf16_bits
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
# (query heads, kv heads, contexts, tree, spoilt node), named for the form that the planner gives them
# (test_attn_plans.py asks it): k_attn_few, or workgroups of 64, 128 and 256 rows with blocks of draft nodes of their
# own or the draft nodes in the merge
DRAFTS = {
    "few64_root": (2, 2, (300,), star(40), 0),
    "own64_root": (8, 2, (300,), star(40), 0),
    "own64_inner": (4, 2, (300,), gen_tree(100, 8, 4, 1), 47),
    "own128_root": (16, 8, (2050,), star(100), 0),
    "own128_inner": (16, 8, (2050,), gen_tree(100, 8, 4, 1), 47),
    "own128_shared_keys_root": (2, 1, (300,), star(40), 0),
    "own256_root": (64, 16, (1000, 300, 0), star(50), 0),
    "own256_inner": (32, 16, (4100,), gen_tree(100, 8, 4, 1), 47),
    "merge64_root": (16, 8, (600,), star(100), 0),
    "merge128_root": (16, 16, (1000, 300, 0, 77), star(40), 0),
    "merge256_root": (64, 16, (1000, 300, 0, 77), star(40), 0),
}


@pytest.mark.parametrize("paged", [False, True], ids=["dense", "paged"])
@pytest.mark.parametrize("name", list(DRAFTS))
def test_a_spoilt_node_reaches_every_descendant(name, paged):
    """The draft nodes are added up in blocks of 32.  A node with a NaN score that is a row's only ancestor in its
    block must not pass for a block without ancestors."""
    heads, kv_heads, ctx, parents, hit = DRAFTS[name]
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
    case = synthetic_case(TB.with_(n_q_heads=heads, n_kv_heads=kv_heads), 700 + len(name), ctx, [parents] * len(ctx))
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


# (query heads, kv heads, nodes, contexts, first keys that are NaN: whole splits of the context, none in part)
CONTEXTS = {
    "few32": (4, 2, 9, (600,), 128),
    "few64": (4, 2, 25, (600,), 128),
    "own64": (4, 2, 100, (600,), 256),
    "own128": (16, 8, 100, (2050,), 256),
    "own128_shared_keys": (2, 1, 40, (300,), 128),
    "own256": (64, 16, 50, (1000, 600, 513), 384),
    "merge64": (16, 8, 100, (600,), 128),
    "merge128": (16, 16, 40, (1000, 600, 700, 513), 256),
    "merge256": (64, 16, 37, (1000, 600, 700, 513), 256),
}


@pytest.mark.parametrize("paged", [False, True], ids=["dense", "paged"])
@pytest.mark.parametrize("name", list(CONTEXTS))
def test_a_stretch_of_spoilt_context_is_not_skipped(name, paged):
    """Keys that are all NaN over exactly one split of the context must not pass for a split without keys."""
    heads, kv_heads, nodes, ctx, spoilt = CONTEXTS[name]
    case = synthetic_case(TB.with_(n_q_heads=heads, n_kv_heads=kv_heads), 800 + len(name), ctx, [gen_tree(nodes, 8, 4, 3)] * len(ctx))
    for k in case.k_ctx:
        k[:, :, :spoilt] = np.nan
    got = case.run_gpu(0.0, paged=paged)["logits"]
    assert not np.isfinite(got).any()


# ------------------------------------------------------------------ logit statistics
# the kernels that end in the LM head's statistics: (batch, nodes, hidden)
HEADS = {"chunks": (1, 40, 256), "ragged_k": (1, 40, 192), "wide": (3, 40, 256)}


def head_case(name):
    batch, nodes, hidden = HEADS[name]
    shape = TB.with_(hidden=hidden, lm_head_std=0.3)
    return synthetic_case(shape, 900 + len(name), (20,) * batch, [gen_tree(nodes, 8, 4, 5 + b) for b in range(batch)])


def with_head_row(case, col, row):
    ws = WeightSource(case.shape, case.seed)

    def get(name, layer):
        bits = ws.bits(name, layer)
        if name == "lm_head":
            bits[col] = np.where(np.isnan(row), np.uint16(0x7FC0), bf16_bits(row))
        return bits
    return model_from_arrays(case.shape, get)


def statistics(logits):
    """fp64; one +inf logit takes all of the probability."""
    x = logits.astype(np.float64)
    top = x.max(axis=-1, keepdims=True)
    with np.errstate(invalid="ignore"):
        d = np.where(x == top, 0.0, x - top)
    e = np.exp(d)
    s = e.sum(axis=-1)
    second = np.sort(e, axis=-1)[:, -2]
    ent = np.log(s) - np.where(e > 0, e * np.where(e > 0, d, 0.0), 0.0).sum(axis=-1) / s
    return x.argmax(axis=-1), 1.0 / s, (1.0 - second) / s, ent


def check_statistics(gpu):
    logits = gpu["logits"].reshape(-1, gpu["logits"].shape[-1])
    arg, conf, margin, ent = statistics(logits)
    assert np.array_equal(gpu["argmax"].reshape(-1), arg)
    # 600 fp32 terms; exp of a distance d carries its rounding, |d| 2^-24: far below 1e-5
    assert np.abs(gpu["confidence"].reshape(-1) - conf).max() <= 1e-5
    assert np.abs(gpu["margin"].reshape(-1) - margin).max() <= 1e-5
    near = np.abs(logits[:, 301]) < 1e30         # beyond, the entropy's sum of p * distance may overflow
    assert np.abs(gpu["entropy"].reshape(-1) - ent)[near].max(initial=0.0) <= 1e-4


def spiked(name, target):
    """One vocabulary entry reads one feature only, with a weight that takes its logit to `target` at the node
    where that feature is largest and to everything between -|target| and |target| at the others."""
    case = head_case(name)
    clean = case.run_gpu(0.0, export_hidden=True)["hidden"].reshape(-1, case.shape.hidden)
    feat = int(np.abs(clean).max(axis=0).argmax())
    peak = clean[np.abs(clean[:, feat]).argmax(), feat]
    row = np.zeros(case.shape.hidden, dtype=np.float32)
    row[feat] = target / float(peak)
    return case.run_gpu(0.0, model=with_head_row(case, 301, row))


@pytest.mark.parametrize("target", [3.1e38, -3.1e38])
@pytest.mark.parametrize("name", list(HEADS))
def test_statistics_of_logits_near_the_end_of_the_range(name, target):
    """exp of a distance beyond 2.4e38 is 0, not a NaN."""
    got = spiked(name, target)
    x = got["logits"][..., 301]
    assert np.isfinite(x).all() and (np.sign(target) * x).max() > 2.5e38
    check_statistics(got)


@pytest.mark.parametrize("name", list(HEADS))
def test_statistics_of_one_infinite_logit(name):
    """It takes all of the probability: confidence and margin 1."""
    got = spiked(name, 8e38)
    x = got["logits"][..., 301].reshape(-1)
    top = x == np.inf
    assert top.any()
    check_statistics(got)
    assert np.all(got["confidence"].reshape(-1)[top] == 1.0) and np.all(got["margin"].reshape(-1)[top] == 1.0)


@pytest.mark.parametrize("name", list(HEADS))
def test_a_nan_logit_does_not_stand_for_the_second_largest(name):
    case = head_case(name)
    top = case.run_gpu(0.0)["argmax"].reshape(-1)
    col = next(int(c) + 1 for c in top if c % 16 < 15 and c + 1 not in top)   # the same thread's, after a largest
    got = case.run_gpu(0.0, model=with_head_row(case, col, np.full(case.shape.hidden, np.nan)))
    x = got["logits"].reshape(-1, case.shape.vocab)
    assert np.isnan(x[:, col]).all()
    rest = np.sort(np.delete(x, col, axis=1), axis=1)
    l1, l2 = (got["_ver"].region(r).view(torch.float32)[:len(x)].cpu().numpy() for r in ("node_l1", "node_l2"))
    assert np.array_equal(l1, rest[:, -1]) and np.array_equal(l2, rest[:, -2])
    assert np.isnan(got["confidence"]).all()


@pytest.mark.parametrize("name", list(HEADS) + ["fp32"])
def test_a_row_of_nan_logits_is_not_trusted(name):
    if name == "fp32":
        case = synthetic_case(SHAPES["tiny"].with_(n_layers=1, vocab=600), 950, (20,), [gen_tree(40, 8, 4, 5)])
    else:
        case = head_case(name)
    model = device_model(case.shape, case.seed)
    bad = case.shape.vocab - 1
    model.tensors["embed"][bad].fill_(float("nan"))
    case.tokens[:, 0] = bad                      # the root: every row
    got = case.run_gpu(0.0, CRIT_TOP1, model=model)
    assert np.isnan(got["logits"]).all()
    assert np.isnan(got["confidence"]).all() and np.isnan(got["margin"]).all() and np.isnan(got["entropy"]).all()
    assert np.all(got["escalate"] == 1) and np.all(got["token"] == -1) and np.all(got["accepted_len"] == 0)
