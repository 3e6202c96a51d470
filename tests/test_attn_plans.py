"""How attention divides rows and keys (plan_attn in csrc/plan.hpp), asked for on the host: the splits cover the keys and start
where the kernels need it, and the GPU cases of test_gpu_attn_forms.py reach every form."""
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


def test_the_gpu_cases_reach_every_form(plans):
    shapes, names = [], []
    for name, (shape, batch, nodes, ctx, kind) in FORMS.items():
        for paged in (0, 1):
            par = parents_of(kind, nodes, 0)
            depth = np.zeros(nodes, dtype=int)
            for i in range(nodes):
                depth[i] = 1 if par[i] < 0 else depth[par[i]] + 1
            shapes.append((batch, shape.n_kv_heads, shape.n_q_heads // shape.n_kv_heads, shape.head_dim, nodes, depth.max(), max(ctx), paged))
            names.append(name)
    seen = set()
    for n, s, p in zip(names, shapes, plans(shapes)):
        assert not p.few, (n, p)
        kg = 1 if p.rows == 256 else (4 if s[2] * s[4] <= 64 or p.rows == 64 else (2 if s[2] * s[4] <= 96 else 1))
        seen.add((p.rows, kg, p.mode, s[3]))
        print(n, s, p)
    for form in ((64, 4), (128, 1), (128, 2), (256, 1)):
        for mode in (IN_MERGE, OWN):
            assert any(f[:3] == (*form, mode) for f in seen), (form, mode, sorted(seen))
    assert {f[3] for f in seen} == {64, 128}
