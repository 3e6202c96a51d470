"""How attention divides rows and keys (plan_attn in csrc/plan.hpp), asked for on the host: the splits cover the keys and start
where the kernels need it, and the GPU cases of the other files take the forms that they are there for."""
import collections
import os
import random
import shutil
import subprocess

import numpy as np
import pytest

from paper_2601_23180_amd import build as B
from test_gpu_attn_forms import FORMS, parents_of

HERE = os.path.dirname(os.path.abspath(__file__))
pytestmark = pytest.mark.skipif(shutil.which(B.HIPCC) is None, reason="no hipcc")
Plan = collections.namedtuple("Plan", "few rows groups keys splits mode blocks")
IN_MERGE, OWN = 0, 1


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    exe = str(tmp_path_factory.mktemp("plans") / "attn_report")
    r = subprocess.run([B.HIPCC, "-O1", *[f for f in B.FLAGS if f != "-O3"], "--cuda-host-only", "-o", exe,
                        os.path.join(HERE, "plans", "attn_report.cpp")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]

    def ask(shapes):
        text = "\n".join(" ".join(str(int(x)) for x in s) for s in shapes)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.splitlines()
        assert len(out) == len(shapes)
        return [Plan(*map(int, line.split())) for line in out]
    return ask


def test_splits_cover_the_keys(plans):
    rng = random.Random(3)
    shapes = []
    while len(shapes) < 4000:
        group, batch = rng.randint(1, 8), rng.randint(1, 8)
        nodes = rng.randint(1, min(128, 512 // group, 256 // batch))
        keys = rng.choice([0, 1, 127, 128, 129, rng.randint(0, 600), rng.randint(0, 20000), rng.randint(0, 140000)])
        shapes.append((batch, rng.randint(1, 32), group, rng.choice([64, 128]), nodes, rng.randint(1, nodes), keys, rng.random() < 0.4))
    for s, p in zip(shapes, plans(shapes)):
        batch, n_kv, group, d, nodes, depth, keys, paged = s
        rows = group * nodes
        assert 1 <= p.splits <= 64 and p.splits * p.keys >= keys and (p.splits == 1 or (p.splits - 1) * p.keys < keys), (s, p)
        assert p.keys % (64 if p.rows == 256 and not paged else 128) == 0 and p.keys >= 128, (s, p)
        assert p.groups == -(-rows // p.rows) and p.rows in ((32, 64) if p.few else (64, 128, 256)), (s, p)
        assert not p.few or p.groups == 1, (s, p)
        assert p.blocks == (0 if p.mode == IN_MERGE else -(-nodes // 32)), (s, p)
        if p.mode == OWN and not p.few:   # one round: a second one costs more than the merge's own draft part
            assert (p.splits + p.blocks) * batch * n_kv * p.groups <= 256, (s, p)


def key_groups(p, rows):
    """Groups of wavefronts among which a workgroup shares the keys of a tile out (launch_attn_bf16_d)."""
    return 1 if p.rows == 256 else (4 if rows <= 64 or p.rows == 64 else (2 if rows <= 96 else 1))


def depth_of(parents):
    depth = np.zeros(len(parents), dtype=int)
    for i, p in enumerate(parents):
        depth[i] = 1 if p < 0 else depth[p] + 1
    return depth.max()


def ask_both(plans, heads, kv_heads, head_dim, trees, ctx):
    """The plans over a contiguous and over a paged cache."""
    depth = max(depth_of(t) for t in trees)
    return plans([(len(ctx), kv_heads, heads // kv_heads, head_dim, len(trees[0]), depth, max(ctx), paged) for paged in (0, 1)])


def form(p):
    return "%s%d" % ("few" if p.few else "merge" if p.mode == IN_MERGE else "own", p.rows)


def test_the_form_chosen_is_about_the_fastest_measured(plans):
    """tests/plans/attn_measured.txt: 151 shapes in up to 22 forms each.  Medians of the same form differ by up to 3 % from run to run."""
    with open(os.path.join(HERE, "plans", "attn_measured.txt")) as f:
        lines = [line.split("|") for line in f if not line.startswith("#")]
    shapes = [tuple(map(int, a.split())) + (0,) for a, _ in lines]
    over = []
    for s, p, (_, forms) in zip(shapes, plans(shapes), lines):
        us, before = {}, None
        for name, t in zip(*[iter(forms.split())] * 2):
            us[name.rstrip("*")] = sum(map(float, t.split("+")))
            before = us[name.rstrip("*")] if name.endswith("*") else before
        mine = us["%dx%d" % (p.rows, p.splits)]   # a form that is not in the file has to be measured first
        over.append(mine / min(us.values()) - 1)
        assert over[-1] < 0.08 and (before is None or mine < 1.03 * before), (s, p, us)
    assert np.mean(over) < 0.006, np.mean(over)


def test_the_gpu_cases_reach_every_form(plans):
    seen = set()
    for name, (shape, batch, nodes, ctx, kind) in FORMS.items():
        for p in ask_both(plans, shape.n_q_heads, shape.n_kv_heads, shape.head_dim, [parents_of(kind, nodes, b) for b in range(batch)], ctx):
            assert form(p) == name.split("_")[0], (name, p)
            seen.add((p.rows, key_groups(p, shape.n_q_heads // shape.n_kv_heads * nodes), p.mode, shape.head_dim))
    for rows_groups in ((64, 4), (128, 1), (128, 2), (256, 1)):
        for mode in (IN_MERGE, OWN):
            assert any(f[:3] == (*rows_groups, mode) for f in seen), (rows_groups, mode, sorted(seen))
    assert {f[3] for f in seen} == {64, 128}


def test_cases_that_are_not_finite_take_the_form_that_they_name(plans):
    from test_gpu_nonfinite import CONTEXTS, DRAFTS
    from workloads import gen_tree
    named = set()
    for name, (heads, kv_heads, ctx, parents, _) in DRAFTS.items():
        for p in ask_both(plans, heads, kv_heads, 128, [parents], ctx):
            assert form(p) == name.split("_")[0], (name, p)
            assert ("shared_keys" in name) == (p.rows == 128 and key_groups(p, heads // kv_heads * len(parents)) == 2), (name, p)
        named.add(name.split("_")[0])
    assert named == {"few64", "own64", "own128", "own256", "merge64", "merge128", "merge256"}
    for name, (heads, kv_heads, nodes, ctx, spoilt) in CONTEXTS.items():
        for p in ask_both(plans, heads, kv_heads, 128, [gen_tree(nodes, 8, 4, 3)], ctx):
            assert form(p) == name.split("_")[0], (name, p)
            assert spoilt % p.keys == 0 and spoilt <= min(ctx) and p.splits > 1, (name, p)   # whole splits
    assert {n.split("_")[0] for n in CONTEXTS} == named | {"few32"}


@pytest.mark.parametrize("head_dim", [64, 128])
def test_the_cases_of_the_reference_of_the_exponents(plans, head_dim):
    import test_gpu_attention_reference as ref
    from workloads import gen_tree
    kinds = set()
    for name, (nodes, heads, kv_heads, ctx, rows, tile, groups, keys) in ref.FORMS.items():
        star = np.array([-1] + [0] * (nodes - 1))
        for seed in (1200, 1400):
            for trees in ([gen_tree(nodes, 8, 4, seed + len(name) + b) for b in range(len(ctx))], [star]):
                for p in ask_both(plans, heads, kv_heads, head_dim, trees, ctx):
                    assert not p.few and (p.rows, p.keys) == (rows, keys), (name, p)
                    assert groups == key_groups(p, heads // kv_heads * nodes) and tile == (64 if p.rows == 256 else 128), (name, p)
                    assert keys >= 2 * tile, name   # a later tile can outgrow the first
        kinds.add((rows, groups, heads // kv_heads * nodes <= 32))
    assert kinds == {(128, 4, True), (128, 4, False), (128, 2, False), (128, 1, False), (64, 4, False), (256, 1, False)}


def test_the_cases_of_long_contexts_and_draft_blocks(plans):
    from test_gpu_parity import LONG
    from test_gpu_tiles import ATTN_CASES
    from workloads import gen_tree
    got = {n: ask_both(plans, heads, kv, 128, [gen_tree(nodes, 8, 4, 33 + b) for b in range(len(ctx))], ctx)
           for n, (ctx, nodes, heads, kv) in LONG.items()}
    assert got["ctx40000"][0][3:5] == (768, 53) and got["ctx1000"][0].keys == 128
    for name, p in got.items():
        rows = [128 if name == "ctx1000" else 64] * 2
        if "kv8" in name:
            rows = [128 if name == "ctx7000_rows240_kv8" else 256] * 2
        elif "rows512" in name:
            rows = [128, 128]
        assert [p[0].rows, p[1].rows] == rows, (name, p)
    assert got["ctx6400_nodes128_rows512_kv8"][0].keys == 448
    for name, (batch, nodes, heads, kv, ctx) in ATTN_CASES.items():
        tree = np.arange(-1, nodes - 1) if nodes == 128 else gen_tree(nodes, 8, 4, 500 + len(name)) if nodes > 1 else np.array([-1])
        for p in ask_both(plans, heads, kv, 128, [tree], ctx):
            assert ("in_merge" in name) == (p.mode == IN_MERGE), (name, p)
            assert "shared_keys" not in name or (not p.few and key_groups(p, heads // kv * nodes) > 1), (name, p)
