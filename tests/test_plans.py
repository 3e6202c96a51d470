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
Plan = collections.namedtuple("Plan", "kernel width tiles splits counters floats built meets apart")


def host_program(tmp_path_factory, name):
    exe = str(tmp_path_factory.mktemp("plans") / name)
    r = subprocess.run([B.HIPCC, "-O1", *[f for f in B.FLAGS if f != "-O3"], "--cuda-host-only", "-o", exe,
                        os.path.join(HERE, "plans", name + ".cpp")], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-3000:]
    return exe


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    """Plans of a list of (epilogue, columns, k, rows, head_dim, qk_norm)."""
    exe = host_program(tmp_path_factory, "plan_report")

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


def test_every_pass_of_the_head_kernel_has_sub_tiles(plans):
    """Over at most 32 rows its workgroups share the sub-tiles of 32 columns out as evenly as integers go, then their
    passes those of a workgroup: one to four sub-tiles each."""
    cols = [*range(1, 2000, 13), 65504, 65505, 65536, 65537, 98304, 98305, 131072, 131073, 151936, 262144, 999999]
    for n, p in zip(cols, plans([(HEAD, n, 512, 9, 128, 0) for n in cols])):
        places, sub, passes = p.tiles // p.splits, (n + 31) // 32, p.splits
        assert p.kernel == HEADK and places * passes == p.tiles
        runs = [sub * (w + 1) // places - sub * w // places for w in range(places)]
        sizes = [r * (i + 1) // passes - r * i // passes for r in set(runs) for i in range(passes)]
        assert sum(runs) == sub and min(sizes) >= 1 and max(sizes) <= 4, (n, p)


def layer_products(batch, nodes, s):
    rows, qd = batch * nodes, s.n_q_heads * s.head_dim
    return [(QKV, qd + 2 * s.n_kv_heads * s.head_dim, s.hidden, rows, s.head_dim, s.qk_norm),
            (RESID, s.hidden, qd, rows, s.head_dim, 0), (SWIGLU, 2 * s.ffn, s.hidden, rows, s.head_dim, 0),
            (RESID, s.hidden, s.ffn, rows, s.head_dim, 0)]


def test_the_gpu_cases_reach_every_width(plans):
    """test_gpu_tiles.py: (product, width, row blocks, several splits) of the streaming kernel."""
    from test_gpu_tiles import CASES
    shapes = [p for _, batch, nodes, shape in CASES for p in layer_products(batch, nodes, shape)]
    got = set()
    for s, p in zip(shapes, plans(shapes)):
        if p.kernel == STREAM:
            got.add((s[0], p.width, rows_laid_out(RESID, p, s[3]) // 16, p.splits > 1))
    every = (1, 2, 3, 4, 6, 8)
    want = {(SWIGLU, w, rb, False) for w in (32, 48, 64, 96, 112) for rb in every if w < 112 or rb <= 4}
    want |= {(RESID, w, rb, sp) for w in (16, 32, 64) for rb in every for sp in (False, True)}
    want |= {(RESID, 128, rb, False) for rb in (1, 2, 3, 4)}      # in splits: products of more than 100M weights
    # 64 columns over 8 row blocks lose to two groups of 4 in 128, but for layers of 17 and more kv heads
    want |= {(QKV, w, rb, sp) for w in (16, 32, 64, 128) for rb in every for sp in (False, True) if (w, rb) != (64, 8)}
    want |= {(QKV, 96, 4, True)}                                  # others: products of more than 40M weights
    assert not want - got, sorted(want - got)


def finishes(shapes, got):
    """(product, width, row blocks of a tile, one split or who finishes the splits) of the streaming kernel."""
    for s, p in zip(shapes, got):
        if p.kernel == STREAM and s[0] in (QKV, RESID, PLAIN):
            groups = p.counters // p.tiles
            rb = 4 if groups > 1 else rows_laid_out(RESID, p, s[3]) // 16
            assert p.meets == (rb >= 3 and p.splits >= rb), (s, p)
            yield s[0], p.width, rb, "together" if p.meets else "one split" if p.splits == 1 else "alone"


def meet_cases():
    """The products of every case of test_gpu_meet.py."""
    from test_gpu_meet import SIZES
    from workloads import SHAPES
    return [layer_products(batch, nodes, SHAPES["tiny_bf16"].with_(hidden=hidden, n_q_heads=nq, n_kv_heads=nkv, head_dim=d, ffn=ffn,
                                                                   qk_norm=bool(norm)))
            for batch, nodes, hidden, nq, nkv, d, ffn, norm in SIZES]


def test_the_gpu_cases_finish_tiles_every_way(plans):
    """test_gpu_tiles.py and test_gpu_meet.py, tiles of three row blocks and more: in one split, several that one workgroup
    finishes, several that all of them finish."""
    from test_gpu_tiles import ADAPTERS, CASES
    shapes = [p for _, batch, nodes, shape in CASES for p in layer_products(batch, nodes, shape)] + sum(meet_cases(), [])
    shapes += [(PLAIN, dim, hidden, batch * nodes, 128, 0) for batch, nodes, hidden, dim in ADAPTERS.values()]
    got = set(finishes(shapes, plans(shapes)))
    ways = ("one split", "alone", "together")
    want = {(epi, w, rb, way) for way in ways for rb in (3, 4, 6, 8) for epi, w in ((QKV, 16), (QKV, 32), (QKV, 64), (QKV, 96), (QKV, 128),
            (RESID, 16), (RESID, 32), (RESID, 64), (PLAIN, 32)) if w < 96 or rb <= 4}
    # never planned for products of up to 30M weights
    want -= {(QKV, 64, 8, "one split"), (QKV, 64, 8, "alone"), (RESID, 64, 3, "alone")}
    assert not want - got, sorted(want - got)


def test_the_gpu_cases_that_meet(plans):
    """test_gpu_meet.py: products of every case are finished by all workgroups of a tile, over every number of row blocks."""
    seen = set()
    for shapes in meet_cases():
        meet = {(f[0], f[2]) for f in finishes(shapes, plans(shapes)) if f[3] == "together"}
        assert meet, shapes
        seen |= meet
    assert seen == {(epi, rb) for epi in (QKV, RESID) for rb in (3, 4, 6, 8)}, sorted(seen)


def test_no_share_of_a_tile_is_taken_twice_or_not_at_all(tmp_path_factory):
    """meet_splits through every order of the steps of two to four workgroups, random ones of up to 16, workgroups leaving
    early or not: the program ends with a message where a share is not taken exactly once, after all have arrived."""
    r = subprocess.run([host_program(tmp_path_factory, "meet_orders")], capture_output=True, text=True)
    assert r.returncode == 0, r.stdout
    orders, departures, takeovers = map(int, r.stdout.split())
    assert orders > 200000 and departures >= takeovers > 10000


def test_the_gpu_cases_of_the_adapter(plans):
    """What the cases of test_gpu_tiles.py are named for."""
    from test_gpu_tiles import ADAPTERS, TB
    planned = {n: plans([(PLAIN, dim, hidden, batch * nodes, 128, 0)])[0]
               for n, (batch, nodes, hidden, dim) in ADAPTERS.items()}
    layers = layer_products(1, 1, TB.with_(hidden=ADAPTERS["rows64_no_counters"][2], ffn=256))
    counters = max(p.counters for rows in (16, 32, 48, 64, 96, 128)
                   for p in plans([(s[0], s[1], s[2], rows, s[4], s[5]) for s in layers]) if p.kernel == STREAM)
    for name, p in planned.items():
        if p.kernel == STREAM and name != "rows64_no_counters":
            assert ("meet" in name) == bool(p.meets) and ("one_split" in name) == (p.splits == 1), (name, p)
    p = planned["rows64_no_counters"]
    assert p.kernel == STREAM and p.splits > 1 and p.tiles > counters
    for name in ("rows23_splits", "rows100_splits_ragged_k"):
        assert planned[name].kernel == STREAM and 1 < planned[name].splits
    assert planned["rows100_one_split"][:2] == (STREAM, 32) and planned["rows100_one_split"].splits == 1
    assert planned["rows250_splits"].kernel == WIDE and planned["rows250_splits"].splits > 1
    assert planned["rows130_one_split"][:2] == (WIDE, 128) and planned["rows130_one_split"].splits == 1
    assert planned["rows130_wide_tiles"][:2] == (WIDE, 256) and planned["rows130_wide_tiles"].splits == 1


def test_row_groups_of_the_head(plans):
    """One after the other where one is all there is, or where a short last one fills the last of several rounds of workgroups and the
    weights are no more than the memory-side cache serves twice; the cases of test_gpu_tiles.py."""
    from test_gpu_tiles import CASES
    named = {c[0]: c for c in CASES if c[0].endswith(("vocab_apart", "vocab_side_by_side"))}
    shapes = [(HEAD, c[3].vocab, c[3].hidden, c[1] * c[2], 128, 0) for c in named.values()]
    shapes += [(HEAD, 50257, 1472, 96, 128, 0), (HEAD, 32768, 4096, 132, 128, 0), (HEAD, 102400, 4096, 192, 128, 0),
               (HEAD, 102400, 4096, 193, 128, 0), (HEAD, 128256, 4096, 132, 128, 0), (HEAD, 36608, 704, 225, 128, 0)]
    got = plans(shapes)
    assert len(named) == 3 and all(p.kernel == WIDE for p in got)
    assert [p.apart for p in got] == [n.endswith("apart") for n in named] + [1, 0, 1, 0, 0, 0]
