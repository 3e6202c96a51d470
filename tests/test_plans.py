"""The plans of the matmuls (csrc/plan.hpp), asked for on the host: they agree with how the kernels lay their
tiles out."""
import collections
import os
import random
import shutil
import subprocess

import pytest

from paper_2601_23180_amd import build as B

HERE = os.path.dirname(os.path.abspath(__file__))
pytestmark = pytest.mark.skipif(shutil.which(B.HIPCC) is None, reason="no hipcc")
QKV, RESID, SWIGLU, HEAD, PLAIN = range(5)
STREAM, HEADK, WIDE = range(3)
Plan = collections.namedtuple("Plan", "kernel width tiles splits counters floats built")


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    """Plans of a list of (epilogue, columns, k, rows, head_dim, qk_norm)."""
    exe = str(tmp_path_factory.mktemp("plans") / "plan_report")
    r = subprocess.run([B.HIPCC, "-O1", *[f for f in B.FLAGS if f != "-O3"], "--cuda-host-only", "-o", exe,
                        os.path.join(HERE, "plans", "plan_report.cpp")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]

    def ask(shapes):
        text = "\n".join(" ".join(str(int(x)) for x in s) for s in shapes)
        out = subprocess.run([exe], input=text, capture_output=True, text=True, check=True).stdout.splitlines()
        assert len(out) == len(shapes)
        return [Plan(*map(int, line.split())) for line in out]
    return ask


def random_shapes(n, seed=7):
    rng = random.Random(seed)
    for _ in range(n):
        d = rng.choice([64, 128])
        kv = rng.randint(1, 16)
        heads = kv * rng.randint(1, 8)
        hidden, ffn, rows = 64 * rng.randint(1, 80), 64 * rng.randint(1, 240), rng.randint(1, 128)
        vocab = rng.choice([129, 50257, 151936, rng.randint(2, 200000)])
        yield [(QKV, (heads + 2 * kv) * d, hidden, rows, d, rng.random() < 0.5), (RESID, hidden, heads * d, rows, d, 0),
               (SWIGLU, 2 * ffn, hidden, rows, d, 0), (RESID, hidden, ffn, rows, d, 0),
               (PLAIN, 4 * rng.randint(1, 2000), hidden, rows, d, 0), (HEAD, vocab, hidden, rows, d, 0)]


def rows_laid_out(epi, plan, rows):
    """Rows of a partial tile, all row groups: whole row blocks of 16 (1 to 4, 6 or 8), or two groups of 64 where a head
    of 128 stays whole."""
    if rows > 64:
        return 128 if rows > 96 or (epi == QKV and plan.width == 128) else 96
    return (rows + 15) // 16 * 16


def test_partial_tiles_are_counted_as_the_kernel_lays_them_out(plans):
    shapes = [s for group in random_shapes(400) for s in group]
    seen = 0
    for s, p in zip(shapes, plans(shapes)):
        if p.kernel == STREAM and p.splits > 1:
            seen += s[0] == QKV and p.width == 128 and 64 < s[3] <= 96
            assert p.floats == p.splits * p.tiles * p.width * rows_laid_out(s[0], p, s[3]), (s, p)
        if p.kernel == STREAM:
            assert p.counters == p.tiles * (2 if s[0] == QKV and p.width == 128 and s[3] > 64 else 1)
    assert seen > 5


def test_every_plan_has_a_kernel(plans):
    """The streaming kernel in a width that it is built in; the 128-column kernel where the reduction has whole chunk
    pairs; the wide kernel for the LM head in 256-column tiles only."""
    shapes = [s for group in random_shapes(1500, seed=8) for s in group]
    for s, p in zip(shapes, plans(shapes)):
        epi, _, k, rows = s[:4]
        if p.kernel == STREAM:
            assert p.built and (epi != HEAD or rows <= 64), (s, p)
        elif p.kernel == HEADK:
            assert epi == HEAD and k % (512 if rows <= 32 else 256) == 0, (s, p)
        else:
            assert p.kernel == WIDE and epi == HEAD and rows > 64 and p.width == 256, (s, p)
