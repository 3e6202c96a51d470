"""The work that a program built on this library has it do, as cases to be timed.

Every model pass goes through `Verifier.verify` (one tree or chain of draft nodes against a KV cache),
a temperature > 0 step through `Verifier.verify` + `SampleDecider.decide`, and a stretch of two-level
decoding through `TernaryDecoder.round`, as a serving loop calls them.  Inputs are seeded noise of the
shapes and distributions that the paths meet: weights N(0, 0.02^2), norm weights around 1, an LM head
scaled so that top-1 probabilities spread, N(0, 1) caches, uniform tokens, random draft trees.
"""
import numpy as np
import torch

from paper_2601_23180_amd import (CRIT_MARGIN, RESAMPLE_RESIDUAL, TRISPEC_BF16, TRISPEC_F32, KVCache, Model,
                                  PagedKVCache, SampleDecider, TernaryDecoder, Verifier)

# layers, hidden, query heads, kv heads, head_dim, ffn, vocabulary, storage type, rotary base, spread of the logits
MODELS = {
    "tiny_f32": (2, 256, 4, 2, 64, 512, 4096, "f32", 1e4, 6.5),
    "odd_width": (12, 1472, 12, 4, 64, 4032, 50257, "bf16", 1e4, 8.5),
    "qwen3_0p6b": (28, 1024, 16, 8, 128, 3072, 151936, "bf16", 1e6, 9.5),
    "qwen3_1p7b": (28, 2048, 16, 8, 128, 6144, 151936, "bf16", 1e6, 9.5),
    "qwen3_8b": (36, 4096, 32, 8, 128, 12288, 151936, "bf16", 1e6, 9.5),
    "llama3_8b": (32, 4096, 32, 8, 128, 14336, 128256, "bf16", 5e5, 9.5),
}
ADAPTER_DIM = 1024    # width of the feature space that the adapter maps to


def _case(name, **kw):
    c = dict(kind="verify", model="", batch=1, nodes=1, ctx=0, tree="chain", paged=False, qk_norm=False,
             features=False, lam=0.5, rounds=0, proxy="")
    c.update(kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest pass: a toy-sized fp32 model, 8 drafts; launches and latency are all of it
        _case("tiny_f32_chain9", model="tiny_f32", nodes=9, ctx=128),
        # a small proxy checks 8 drafted tokens
        _case("0p6b_chain9", model="qwen3_0p6b", nodes=9, ctx=2048),
        # the proxy of the two-level scheme over a full draft tree and a long context
        _case("1p7b_tree60_ctx8k", model="qwen3_1p7b", nodes=60, ctx=8192, tree="tree"),
        # the target over a full draft tree: the benchmark's default workload
        _case("8b_tree60_ctx4k", model="qwen3_8b", nodes=60, ctx=4096, tree="tree"),
        # plain decoding with the target: one token (a round without drafts, a one-token lag)
        _case("8b_single", model="qwen3_8b", nodes=1, ctx=1500, lam=0.0),
        # taking in a prompt: a chain of as many tokens as one pass holds
        _case("8b_prompt128", model="qwen3_8b", nodes=128, ctx=1024, lam=0.0),
        # four sequences at once, long reasoning contexts
        _case("8b_b4_tree60_ctx16k", model="llama3_8b", batch=4, nodes=60, ctx=16384, tree="tree"),
        # a serving mix: paged cache, unequal contexts, per-head norms, features and adapter for the drafter
        _case("1p7b_paged_b3_tree37", model="qwen3_1p7b", batch=3, nodes=37, ctx=3001, tree="tree", paged=True,
              qk_norm=True, features=True),
        # widths that are multiples of 64 only, head_dim 64, a vocabulary that fills no tile
        _case("odd_width_b2_tree23", model="odd_width", batch=2, nodes=23, ctx=777, tree="tree"),
        # temperature > 0: pass, then acceptance and the residual draw, four chains at once
        _case("0p6b_sample_b4", kind="sample", model="qwen3_0p6b", batch=4, nodes=9, ctx=2048, lam=0.0),
        # a stretch of two-level decoding in its lossless setting (threshold above 1): every round runs
        # proxy and target, commits both caches and comes back to the host
        _case("ternary_1p7b_8b", kind="rounds", model="qwen3_8b", proxy="qwen3_1p7b", nodes=60, ctx=8192,
              tree="tree", lam=1.5, rounds=4),
    ]


def _log_int(rng, lo, hi):
    return int(round(np.exp(rng.uniform(np.log(lo), np.log(hi)))))


def draw(rng):
    kind = rng.choice(["verify", "verify", "verify", "verify", "sample", "rounds"])
    tree = "chain" if kind == "sample" else rng.choice(["chain", "tree"])
    if kind == "rounds":
        proxy, model = rng.choice([("qwen3_0p6b", "qwen3_1p7b"), ("qwen3_0p6b", "qwen3_8b"), ("qwen3_1p7b", "qwen3_8b")])
        return _case("", kind=kind, model=model, proxy=proxy, nodes=_log_int(rng, 2, 60), ctx=_log_int(rng, 64, 8192),
                     tree=tree, lam=rng.choice([0.0, 1.5]), rounds=rng.randint(1, 3))
    model = rng.choice(sorted(MODELS))
    group = MODELS[model][2] // MODELS[model][3]
    if kind == "sample":
        batch = rng.randint(1, 4)
        return _case("", kind=kind, model=model, batch=batch, nodes=_log_int(rng, 1, 16), ctx=_log_int(rng, 16, 4096),
                     qk_norm=rng.random() < 0.5, lam=0.0)
    batch = rng.choice([1, 1, 1, 2, 3, 4])
    nodes = _log_int(rng, 1, min(128, 256 // batch, 512 // group))
    longest = 2048 if model == "tiny_f32" else 16384 if MODELS[model][1] < 4096 or batch > 1 else 8192
    return _case("", model=model, batch=batch, nodes=nodes, ctx=_log_int(rng, 16, longest), tree=tree,
                 paged=rng.random() < 0.3, qk_norm=rng.random() < 0.5, features=rng.random() < 0.25,
                 lam=rng.choice([0.0, 0.3, 0.5, 0.9]))


def _ctx_lens(case):
    """Context of every sequence: equal, except in paged caches, where sequences come and go."""
    if not case["paged"]:
        return [case["ctx"]] * case["batch"]
    return [max(1, case["ctx"] - 611 * b % max(1, case["ctx"])) for b in range(case["batch"])]


def _model(name, qk_norm, gen):
    layers, hidden, nq, nkv, d, ffn, vocab, dtype, base, spread = MODELS[name]
    dt = torch.float32 if dtype == "f32" else torch.bfloat16

    def mat(rows, cols, std):
        return torch.empty((rows, cols), dtype=dt, device="cuda").normal_(0.0, std, generator=gen)

    def norm(n):
        return torch.empty(n, dtype=torch.float32, device="cuda").normal_(1.0, 0.1, generator=gen).to(dt)

    t = {"embed": mat(vocab, hidden, 0.02), "lm_head": mat(vocab, hidden, spread / hidden ** 0.5),
         "final_norm": norm(hidden)}
    for key, rows, cols in (("wq", nq * d, hidden), ("wk", nkv * d, hidden), ("wv", nkv * d, hidden),
                            ("wo", hidden, nq * d), ("w_gate", ffn, hidden), ("w_up", ffn, hidden),
                            ("w_down", hidden, ffn)):
        t[key] = [mat(rows, cols, 0.02) for _ in range(layers)]
    t["norm_attn"] = [norm(hidden) for _ in range(layers)]
    t["norm_ffn"] = [norm(hidden) for _ in range(layers)]
    if qk_norm:
        t["q_norm"] = [norm(d) for _ in range(layers)]
        t["k_norm"] = [norm(d) for _ in range(layers)]
    m = Model(n_layers=layers, hidden=hidden, n_q_heads=nq, n_kv_heads=nkv, head_dim=d, ffn=ffn, vocab=vocab,
              dtype=TRISPEC_F32 if dtype == "f32" else TRISPEC_BF16, rms_eps=1e-6, rope_base=base, tensors=t,
              qk_norm=qk_norm)
    m.pack(release_originals=True)
    return m


def _tree(kind, n, rng):
    """parents of a chain, or of a tree of depth 8 at most with up to 4 children a node, in level order;
    and the depths."""
    if kind == "chain":
        return np.arange(-1, n - 1, dtype=np.int32), np.arange(n, dtype=np.int32)
    parents, depth, kids = [-1], [0], [0]
    while len(parents) < n:
        i = len(parents)
        room = [j for j in range(i) if depth[j] < 8 and kids[j] < 4]
        p = i - 1 if i <= 8 else int(rng.choice(room))
        parents.append(p); depth.append(depth[p] + 1); kids.append(0); kids[p] += 1
    order = sorted(range(n), key=lambda j: (depth[j], j))
    new = {old: k for k, old in enumerate(order)}
    return (np.array([-1 if parents[j] < 0 else new[parents[j]] for j in order], dtype=np.int32),
            np.array([depth[j] for j in order], dtype=np.int32))


def _new_rows(kv, lens, nodes):
    """Views of the cache slots that a pass appends to (paged: the pages that hold them)."""
    if not hasattr(kv, "table"):
        return [t for b, c in enumerate(lens) for t in (kv.k[:, b, :, c:c + nodes], kv.v[:, b, :, :, c:c + nodes])]
    table, out = kv.table.cpu().numpy(), []
    for b, c in enumerate(lens):
        for p in range(c // 256, (c + nodes - 1) // 256 + 1):
            out += [kv.k_pool[:, int(table[b, p])], kv.v_pool[:, int(table[b, p])]]
    return out


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    rng = np.random.default_rng(seed)
    n, lens = case["nodes"], _ctx_lens(case)
    model = _model(case["model"], case["qk_norm"], gen)
    vocab = model.cfg.vocab
    s = {"case": case, "model": model}

    if case["kind"] == "rounds":
        proxy = _model(case["proxy"], case["qk_norm"], gen)
        grow = (case["rounds"] + 1) * n
        dec = TernaryDecoder(proxy, model, (case["ctx"] + grow + 128 + 63) // 64 * 64, max_nodes=max(64, n))
        for kv in (dec.kv_p, dec.kv_t):
            kv.k.normal_(generator=gen)
            kv.v.normal_(generator=gen)
        rows = [v for kv in (dec.kv_p, dec.kv_t) for v in _new_rows(kv, lens, case["rounds"] * 9)]
        drafts = [(_tree(case["tree"], n, rng)[0].tolist(), rng.integers(0, vocab, n).tolist())
                  for _ in range(case["rounds"])]
        s.update(dec=dec, proxy=proxy, drafts=drafts, rows=rows, seq=rng.integers(0, vocab, case["ctx"] + 1).tolist())
        return s

    cap = (max(lens) + n + 63) // 64 * 64
    kv = PagedKVCache(model, case["batch"], cap, seed=seed) if case["paged"] else KVCache(model, case["batch"], cap)
    for t in ((kv.k_pool, kv.v_pool) if case["paged"] else (kv.k, kv.v)):
        t.normal_(generator=gen)
    kv.set_len(lens)
    trees = [_tree(case["tree"], n, rng) for _ in lens]
    ver = Verifier(model, case["batch"], n, debug_logits=True, export_hidden=case["features"])
    outputs = dict(ver.out, logits=ver.logits, rows=_new_rows(kv, lens, n))
    if case["features"]:
        layers = model.cfg.n_layers
        ver.feature_layers = sorted({layers // 4, layers // 2, layers - 1})
        shape = (len(ver.feature_layers), case["batch"], n, model.cfg.hidden)
        ver.features = torch.zeros(shape, dtype=torch.float32, device="cuda")
        w = torch.empty((ADAPTER_DIM, model.cfg.hidden), dtype=model.tensors["embed"].dtype, device="cuda")
        bias = torch.empty(ADAPTER_DIM, dtype=torch.float32, device="cuda").normal_(generator=gen)
        adapted = ver.set_adapter(w.normal_(0.0, 0.02, generator=gen), bias)
        outputs.update(hidden=ver.hidden, features=ver.features, adapted=adapted)
    s.update(kv=kv, ver=ver, outputs=outputs, parents=np.stack([t[0] for t in trees]),
             tok=torch.from_numpy(rng.integers(0, vocab, (case["batch"], n)).astype(np.int32)).cuda(),
             pos=torch.from_numpy(np.stack([c + t[1] for c, t in zip(lens, trees)]).astype(np.int32)).cuda())
    if case["kind"] == "sample":
        # the drafter's distributions, the tokens drawn from them, the uniforms of acceptance and draw
        f32 = dict(dtype=torch.float32, device="cuda")
        b = case["batch"]
        s["p_draft"] = torch.softmax(torch.empty((b, n - 1, vocab), **f32).normal_(0.0, 9.5, generator=gen), dim=-1)
        if n > 1:
            picks = torch.multinomial(s["p_draft"].reshape(b * (n - 1), vocab), 1, generator=gen)
            s["tok"][:, 1:] = picks.reshape(b, n - 1).to(torch.int32)
        s["u_accept"] = torch.rand((b, n), generator=gen, **f32)
        s["u_sample"] = torch.rand(b, generator=gen, **f32)
        s["sampler"] = SampleDecider(b, n, vocab)
        outputs["sampled"] = s["sampler"].out
    return s


def run(s):
    case = s["case"]
    if case["kind"] == "rounds":
        dec, seen = s["dec"], []
        dec.kv_p.set_len([case["ctx"]])
        dec.kv_t.set_len([case["ctx"]])
        dec.resume(s["seq"])
        for parents, tokens in s["drafts"]:
            rec = dec.round(parents, tokens, case["lam"])
            seen += [rec["escalate"], rec["catch_up"], rec["proxy"]["accepted_len"], rec["proxy"]["token"]]
            if rec["escalate"]:
                seen += [rec["target"]["accepted_len"], rec["target"]["token"]]
        return {"rounds": np.array(seen), "emitted": np.array(dec.seq[case["ctx"] + 1:]), "rows": s["rows"]}
    s["ver"].verify(s["kv"], s["tok"], s["parents"], s["pos"], case["lam"], CRIT_MARGIN)
    if case["kind"] == "sample":
        s["sampler"].decide(s["ver"].logits, s["tok"], s["p_draft"], s["u_accept"], s["u_sample"], 0.8, case["lam"],
                            CRIT_MARGIN, 1, RESAMPLE_RESIDUAL)
    return s["outputs"]


def _pass_work(name, batch, nodes, lens, logits, features=False):
    layers, hidden, nq, nkv, d, ffn, vocab, dtype = MODELS[name][:8]
    size, rows = 4 if dtype == "f32" else 2, batch * nodes
    layer = 2 * hidden * nq * d + 2 * hidden * nkv * d + 3 * hidden * ffn
    weights = layers * (layer + 2 * hidden) + vocab * hidden
    keys = sum(lens) + rows
    read = size * (weights + rows * hidden + layers * 2 * keys * nkv * d)
    written = 4 * rows * (vocab if logits else 0)
    flops = 2 * rows * (layers * layer + vocab * hidden)
    flops += sum(4 * layers * nodes * (c + nodes) * nq * d for c in lens)
    if features:
        read += size * ADAPTER_DIM * hidden
        written += 4 * rows * (4 * hidden + ADAPTER_DIM)
        flops += 2 * rows * ADAPTER_DIM * hidden
    return read + written, flops


def work(case):
    lens, b, n = _ctx_lens(case), case["batch"], case["nodes"]
    if case["kind"] == "rounds":
        passes = [case["proxy"]] + ([case["model"]] if case["lam"] > 1 else [])
        each = [_pass_work(m, b, n, lens, False) for m in passes]
        return {"bytes": case["rounds"] * sum(e[0] for e in each), "flops": case["rounds"] * sum(e[1] for e in each)}
    byts, flops = _pass_work(case["model"], b, n, lens, True, case["features"])
    if case["kind"] == "sample":
        byts += 4 * b * MODELS[case["model"]][6] * (n + 1)   # the logits again, the draft row where the walk stops
    return {"bytes": byts, "flops": flops}


def tolerance(case):
    # Measured against the same pass in float64 and against another order of the k splits: logits 4e-5
    # and statistics up to 2.5e-4 relative (fp32 model: 1e-6); an appended bf16 cache entry may round the
    # other way (one place of 2^-7).  The margin of a lone node is one small difference of two
    # probabilities, up to 2e-3 of itself off.
    few = 5 if case["batch"] * case["nodes"] < 8 else 1
    if case["model"] == "tiny_f32":
        return {"rel": 5e-6 * few, "max": 5e-5 * few, "differ": 0.01}
    return {"rel": 1e-3 * few, "max": 0.02, "differ": 0.01}
