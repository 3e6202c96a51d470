"""Vocabulary statistics and decision in one launch: sizes around what a workgroup reads at once (fp32: 4096 logits,
bf16: 1280 tiles), several sequences, walks through both halves of the node table."""
import numpy as np
import pytest
import torch

from oracle import CRIT_MARGIN, CRIT_TOP1, decide, node_stats
from workloads import SHAPES, gen_draft_tokens, gen_kv_cache, gen_tree, tree_depths
from gpu_helpers import Case

pytestmark = pytest.mark.gpu

# (model, vocabulary, sequences, nodes)
SIZES = {
    "f32_two": ("tiny", 2, 1, 3),
    "f32_255": ("tiny", 255, 2, 40),
    "f32_4096": ("tiny", 4096, 1, 9),
    "f32_4097": ("tiny", 4097, 3, 70),
    "f32_20011": ("tiny", 20011, 1, 128),
    "bf16_tile": ("tiny_bf16", 130, 3, 40),
    "bf16_1281_tiles": ("tiny_bf16", 163968, 1, 70),
    "bf16_wide": ("tiny_bf16", 2001, 2, 128),
}


def make_case(name):
    model, vocab, batch, nodes = SIZES[name]
    shape = SHAPES[model].with_(n_layers=1, vocab=vocab, lm_head_std=0.3)
    k, v = gen_kv_cache(shape, batch, 20, 7, 0)
    trees = [gen_tree(nodes, 8, 4, 11 + b) if nodes > 3 else np.array([-1, 0, 1], dtype=np.int32) for b in range(batch)]
    tokens = [gen_draft_tokens(t, vocab, 11 + b) if vocab > 4 else np.array([0, 1, 1], dtype=np.int32) for b, t in enumerate(trees)]
    return Case(shape, 7, [k[b][None].astype(np.float64) for b in range(batch)], [v[b][None].astype(np.float64) for b in range(batch)],
                np.stack(tokens), np.stack(trees), np.stack([20 + tree_depths(t) for t in trees]))


@pytest.mark.parametrize("name", list(SIZES))
def test_statistics_and_decision_of_the_pass_s_own_logits(name):
    case = make_case(name)
    got = case.run_gpu(0.05, CRIT_TOP1)
    # A term's exponent is off by half a place of its distance to the largest, a few times over (tile, thread, wavefront,
    # row): 4 * 2^-24 * |d| e^d <= 1e-7, and the sum's own roundings are of that size; 4e-6 leaves a factor for
    # the distances of entropies (a sum of e^d d of either size).
    for b in range(case.batch):
        st = node_stats(got["logits"][b])
        assert np.array_equal(got["argmax"][b], st["argmax"])
        np.testing.assert_allclose(got["confidence"][b], st["conf"], rtol=4e-6)
        np.testing.assert_allclose(got["margin"][b], st["margin"], rtol=0, atol=4e-6)
        np.testing.assert_allclose(got["entropy"][b], st["entropy"], rtol=0, atol=4e-5)
    # the decision that the last workgroup took, and the one of a launch of its own
    alone = {k: v.cpu().numpy().copy() for k, v in got["_ver"].decide(got["_tok"], case.parents, 0.05, CRIT_TOP1).items()}
    for key in ("accepted_len", "token", "escalate", "path"):
        assert np.array_equal(got[key], alone[key]), key


@pytest.mark.parametrize("name", ["f32_4097", "bf16_wide", "f32_20011"])
def test_walks_through_all_nodes(name):
    """Drafts that repeat the verifier's own choice, along chains and trees: the walk reaches nodes past the 64th."""
    case = make_case(name)
    nodes = case.n_nodes
    got = case.run_gpu(0.0)
    for parents in (np.arange(-1, nodes - 1, dtype=np.int32), np.array([-1] + [(i - 1) // 2 for i in range(1, nodes)], dtype=np.int32),
                    np.array([-1] + [max(0, i - 3) for i in range(1, nodes)], dtype=np.int32)):
        tokens = np.zeros_like(case.tokens)
        for b in range(case.batch):
            for i in range(1, nodes):
                tokens[b, i] = got["argmax"][b, parents[i]] if i % 5 else (got["argmax"][b, parents[i]] + 1) % case.shape.vocab
            if parents[1] == 0 and parents[2] == 1:
                tokens[b, 1:] = got["argmax"][b, :-1]
        pars = np.stack([parents] * case.batch)
        out = got["_ver"].decide(torch.from_numpy(tokens).cuda(), pars, 0.0, CRIT_MARGIN)
        for b in range(case.batch):
            want = decide(tokens[b], parents, got["argmax"][b], got["confidence"][b], got["margin"][b], 0.0, CRIT_MARGIN, 1)
            assert int(out["accepted_len"][b]) == want["accepted_len"] and int(out["token"][b]) == want["token"]
            assert [int(x) for x in out["path"][b] if x >= 0] == list(want["path"])
        if parents[-1] == nodes - 2:
            assert int(out["accepted_len"][0]) == nodes - 1
