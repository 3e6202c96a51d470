"""The reference that the attention's long loops take exponents against, a running maximum per row: contexts whose
later tiles hold much larger scores than the first for some rows of a wavefront and not for others.  The forms are
those whose wavefronts share the keys of a tile out (four groups of one row block, four of two, two of four), also in
several 64-row workgroups side by side, and the 128-row and 256-row workgroups whose wavefronts see every key."""
import numpy as np
import pytest

from oracle import OracleWeights, verify_forward
from paper_2601_23180_amd import model_from_arrays
from workloads import SHAPES, WeightSource, gen_draft_tokens, gen_kv_cache, gen_tree, tree_depths
from workloads.gen import bf16_bits, bf16_bits_to_f32
from gpu_helpers import Case, device_model
from test_gpu_parity import full_check, logits_ok

pytestmark = pytest.mark.gpu

TB = SHAPES["tiny_bf16"].with_(n_layers=1, vocab=600, lm_head_std=0.2)
MUCH = 8.0   # log2 units
# name: (nodes, query heads, kv heads, contexts, rows of a workgroup, keys of a tile, key groups, keys of a split); splits of two
# tiles and more.  test_attn_plans.py asks the planner for the last four.
FORMS = {
    "rows18": (9, 4, 2, (16500, 300), 128, 128, 4, 512),
    "rows52": (26, 4, 2, (9000, 8001), 128, 128, 4, 256),
    "rows74": (37, 16, 8, (2050, 130), 128, 128, 2, 256),
    "rows100": (50, 32, 16, (600, 513, 130), 128, 128, 1, 256),
    "rows100_kv2": (50, 4, 2, (3001,), 64, 128, 4, 256),
    "rows200": (50, 64, 16, (1000, 600, 130), 256, 64, 1, 384),
}


def context_case(shape, seed, ctx, parents, key_scale=None, v_scale=1.0):
    """Contexts of noise; key_scale: a factor per slot, cycled through in runs of 32 slots."""
    k, v = gen_kv_cache(shape, len(ctx), max(ctx), seed, 0)
    if key_scale is not None:
        scale = np.resize(np.repeat(np.asarray(key_scale, dtype=np.float32), 32), max(ctx))
        k = bf16_bits_to_f32(bf16_bits(k * scale[:, None]))
    return Case(shape, seed, [k[b][None, :, :n].astype(np.float64) for b, n in enumerate(ctx)],
                [v[b][None, :, :n].astype(np.float64) * v_scale for b, n in enumerate(ctx)],
                np.stack([gen_draft_tokens(p, shape.vocab - 1, seed + b) for b, p in enumerate(parents)]),
                np.stack(parents), np.stack([n + tree_depths(p) for n, p in zip(ctx, parents)]))


def queries(case, b=0, get=None):
    """[node, head, feature] after the rotary embedding."""
    trace = []
    verify_forward(OracleWeights(get or WeightSource(case.shape, case.seed).get), case.shape, case.k_ctx[b][:, :, :1],
                   case.v_ctx[b][:, :, :1], case.tokens[b], case.parents[b], case.positions[b], trace=trace)
    return trace[0]["q"]


def outgrown(case, form):
    """Over the wavefronts of the first sequence: how many have a row whose largest score in the second tile of a
    split exceeds that of the first by much, beside a row for which it does not."""
    nodes, heads, kv_heads, ctx, _, kt, groups, kps = FORMS[form]
    q, k, d, per = queries(case), case.k_ctx[0][0], case.shape.head_dim, heads // kv_heads
    found = 0
    for kvh in range(kv_heads):
        rows = np.concatenate([q[:, kvh * per + al] for al in range(per)])   # rows in the kernel's order
        s = rows @ k[kvh].T * (np.log2(np.e) / np.sqrt(d))
        for first in range(0, ctx[0] - 2 * kt, kps):
            for kw in range(0, kt, kt // groups):
                tile = [s[:, first + t * kt + kw:first + t * kt + kw + kt // groups].max(axis=1) for t in (0, 1)]
                grew = tile[1] > tile[0] + MUCH
                found += sum(grew[r:r + 32].any() and not grew[r:r + 32].all() for r in range(0, len(grew), 32))
    return found


GROWTH = {"jumps": (1, 1, 8, 1, 25, 2, 1), "mild": (1, 4, 2, 6, 1, 5, 1)}


@pytest.mark.parametrize("paged", [False, True], ids=["dense", "paged"])
@pytest.mark.parametrize("head_dim", [64, 128])
@pytest.mark.parametrize("growth", list(GROWTH))
@pytest.mark.parametrize("form", list(FORMS))
def test_growing_scores(form, growth, head_dim, paged):
    """Bars of test_gpu_parity.py.  The high + low parts of a query (2^-17 of it) put an error of 2^-17 of the scores'
    spread, at most 20 log2 units, on a score: 1e-4 of a probability, and of a logit of up to 4."""
    nodes, heads, kv_heads, ctx = FORMS[form][:4]
    seed = 1200 + len(form)
    case = context_case(TB.with_(n_q_heads=heads, n_kv_heads=kv_heads, head_dim=head_dim), seed, ctx,
                        [gen_tree(nodes, 8, 4, seed + b) for b in range(len(ctx))], GROWTH[growth])
    assert growth != "jumps" or outgrown(case, form) > 10
    full_check(case, thresholds=(0.0, 0.5), paged=paged)


@pytest.mark.parametrize("form", list(FORMS))
def test_a_node_does_not_depend_on_its_siblings(form):
    """One slot is a key that the query of one child of the root, and no other, is drawn to by 20 log2 units.  That
    child's token changes; every other node's logits stay the same to the last bit."""
    nodes, heads, kv_heads, ctx = FORMS[form][:4]
    star = np.array([-1] + [0] * (nodes - 1), dtype=np.int32)
    case = context_case(TB.with_(n_q_heads=heads, n_kv_heads=kv_heads), 1300, ctx, [star] * len(ctx))
    d, asked = case.shape.head_dim, queries(case)
    for kvh in range(kv_heads):
        q = asked[nodes - 1, kvh * (heads // kv_heads)]
        case.k_ctx[0][0, kvh, 200] = q * (20.0 / np.log2(np.e) * np.sqrt(d) / (q @ q))   # in the second tile of a split
    model = device_model(case.shape, case.seed)
    drawn = case.run_gpu(0.0, model=model)["logits"]
    case.tokens[0][nodes - 1] = case.shape.vocab - 1   # drafted nowhere else
    other = case.run_gpu(0.0, model=model)["logits"]
    assert np.abs(drawn[0, -1] - other[0, -1]).max() > 0.1
    assert np.array_equal(drawn[0, :-1], other[0, :-1])


@pytest.mark.parametrize("form", list(FORMS))
def test_large_values_do_not_overflow(form):
    """Cached values of about 1e37: the sums of probability times value stay in the range of fp32 as long as no
    probability exceeds 1."""
    nodes, heads, kv_heads, ctx = FORMS[form][:4]
    shape, seed = TB.with_(n_q_heads=heads, n_kv_heads=kv_heads), 1400 + len(form)
    case = context_case(shape, seed, ctx, [gen_tree(nodes, 8, 4, seed + b) for b in range(len(ctx))],
                        GROWTH["mild"], v_scale=2.0 ** 123)
    ws = WeightSource(shape, seed)

    def get(name, layer=0):
        w = ws.get(name, layer)
        return w * np.float32(2.0 ** -100) if name == "wo" else w   # exact in bf16

    def bits(name, layer=0):
        w = ws.bits(name, layer)
        return (np.ascontiguousarray(get(name, layer)).view(np.uint32) >> 16).astype(np.uint16) if name == "wo" else w

    got = case.run_gpu(0.0, model=model_from_arrays(shape, bits))
    for b in range(case.batch):
        want = verify_forward(OracleWeights(get), shape, case.k_ctx[b], case.v_ctx[b], case.tokens[b], case.parents[b],
                              case.positions[b])
        logits_ok(shape, got["logits"][b], want["logits"])
