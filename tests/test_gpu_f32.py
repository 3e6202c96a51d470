"""fp32 models: the edges of the matmul's row groups, reductions and columns that no vector load fits, matrices that start
off a 16-byte boundary, and key counts around a workgroup's first sweep and its shares of the values."""
import numpy as np
import pytest
import torch

from paper_2601_23180_amd import Model
from workloads import SHAPES, gen_draft_tokens, gen_kv_cache, gen_tree, tree_depths
from gpu_helpers import Case, compare_decisions, device_model

pytestmark = pytest.mark.gpu

T = SHAPES["tiny"].with_(vocab=515)
ODD = T.with_(hidden=250, ffn=511, vocab=1003)      # 250 % 4, 511 % 4: single elements; an odd number of columns
# (shape, batch, nodes, contexts)
CASES = {
    "rows4": (T, 1, 4, (60,)),
    "rows5": (T, 1, 5, (59,)),
    "rows8_keys63": (T, 1, 8, (55,)),
    "rows9_keys64": (T, 1, 9, (55,)),
    "rows13_empty": (T, 1, 13, (0,)),
    "rows16_keys256": (T, 1, 16, (240,)),
    "rows17_keys257": (T, 1, 17, (240,)),
    "rows34_d128": (T.with_(head_dim=128), 2, 17, (500, 111)),
    "rows128_norms": (T.with_(qk_norm=True), 1, 128, (300,)),
    "rows246": (T, 2, 123, (77, 1029)),
    "odd_rows3": (ODD, 1, 3, (20,)),
    "odd_rows21": (ODD, 3, 7, (20, 0, 128)),
    "odd_norms": (ODD.with_(qk_norm=True, hidden=254), 1, 12, (40,)),
}


def make_case(name):
    shape, batch, nodes, ctx = CASES[name]
    trees = [gen_tree(nodes, 8, 4, 31 + b) for b in range(batch)]
    kv = [gen_kv_cache(shape, batch, max(max(ctx), 1), 31, l) for l in range(shape.n_layers)]
    cut = lambda which, b: np.stack([layer[which][b][:, :ctx[b]] for layer in kv]).astype(np.float64)
    return Case(shape, 31, [cut(0, b) for b in range(batch)], [cut(1, b) for b in range(batch)],
                np.stack([gen_draft_tokens(t, shape.vocab, 31 + b) for b, t in enumerate(trees)]), np.stack(trees),
                np.stack([c + tree_depths(t) for c, t in zip(ctx, trees)]))


def check(case, got):
    want = case.run_oracle()
    for b in range(case.batch):
        # fp32 sums of at most 1157 terms of logits up to about 30: 2^-24 * sqrt(1157) * 30 a layer, 6e-5; the bar of every fp32 test
        assert np.abs(got["logits"][b] - want[b]["logits"]).max() <= 1e-4
    compare_decisions(case, got, want, 0.5, 0)
    return want


@pytest.mark.parametrize("paged", [False, True], ids=["dense", "paged"])
@pytest.mark.parametrize("name", list(CASES))
def test_passes(name, paged):
    case = make_case(name)
    check(case, case.run_gpu(0.5, paged=paged))


@pytest.mark.parametrize("name", ["rows9_keys64", "rows17_keys257"])
def test_matrices_off_a_16_byte_boundary(name):
    case = make_case(name)
    m = device_model(case.shape, case.seed)

    def shifted(t):
        buf = torch.empty(t.numel() + 1, dtype=t.dtype, device=t.device)
        buf[1:] = t.reshape(-1)
        return buf[1:].view(t.shape)
    t = {k: [shifted(x) for x in v] if isinstance(v, list) else shifted(v) for k, v in m.tensors.items()}
    assert t["wq"][0].data_ptr() % 16 == 4
    c = m.cfg
    odd = Model(n_layers=c.n_layers, hidden=c.hidden, n_q_heads=c.n_q_heads, n_kv_heads=c.n_kv_heads, head_dim=c.head_dim,
                ffn=c.ffn, vocab=c.vocab, dtype=c.dtype, rms_eps=c.rms_eps, rope_base=c.rope_base, tensors=t)
    check(case, case.run_gpu(0.5, model=odd))


def test_features_of_an_odd_width():
    case = make_case("odd_rows21")
    got = case.run_gpu(0.5, export_hidden=True)
    want = case.run_oracle()
    head = device_model(case.shape, case.seed).tensors["lm_head"].double().cpu().numpy()
    for b in range(case.batch):   # the exported features give the logits
        np.testing.assert_allclose(got["hidden"][b].reshape(case.n_nodes, -1).astype(np.float64) @ head.T, want[b]["logits"], rtol=0, atol=1e-4)
