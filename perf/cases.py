"""What a user of this library has it do, as timed cases: verification steps of speculative decoding through
the device-resident form, the host-array form and the whole-model step, and the host drafter's side of a
request.  Sizes are those of the benchmark workloads, the decode loop and the tests, and the ranges between.

A case is a dict of plain values.  Steps (`path` "device", "host", "call" or "model"):

  hq, hkv, d      query heads, kv heads, head dimension         dtype, logits   "bf16" / "f32" each
  batch           sequences                                     s_lo, s_hi      range of their cached prefixes
  n_lo, n_hi      range of their tree sizes                     shape_seed      fixes the lengths inside the ranges
  depth           deepest node                                  vocab           vocabulary
  block           0 contiguous cache, else tokens per block     head_major      cache layout
  layers          caches of the step (1 except for "model")     accept          chance that a node's child is accepted

The drafter (`path` "draft"): prompt, steps, budget, depth, ll, fl, lc, fc, vocab, frozen (tokens of the
corpus sample of a frozen table, 0 = none).
"""
import math
import random

import numpy as np
import torch

from paper_2511_21699_amd import binding as B
from paper_2511_21699_amd import workloads as W

_STEP = dict(path="device", hq=32, hkv=32, d=128, dtype="bf16", logits="bf16", batch=1, s_lo=2048, s_hi=2048, n_lo=64, n_hi=64,
             shape_seed=0, depth=6, vocab=32000, block=0, head_major=False, layers=1, accept=0.6)


def _step(name, **kw):
    return dict(_STEP, name=name, **kw)


def listed():
    return [
        # the smallest step: a small fp32 model, where launches are all there is
        _step("tiny_f32", hq=8, hkv=8, d=64, dtype="f32", logits="f32", s_lo=256, s_hi=256, n_lo=15, n_hi=15, depth=4, vocab=1000),
        # the beginning of an interactive request: short prefix, a tree of the size the drafter finds on
        # average, results needed on the host to draft the next one
        _step("host_short", path="host", s_lo=300, s_hi=300, n_lo=16, n_hi=16),
        # the same request later on: the decode loop's mean prefix, the full node budget, an odd size
        _step("host_decode", path="host", s_lo=4111, s_hi=4111, n_lo=63, n_hi=63),
        # the benchmark's headline shape
        _step("mha_2k"),
        # one call with everything marshalled on the spot, as a script or a test makes it; head_dim 64 with
        # grouped queries and a large vocabulary with fp32 logits, as small models have them
        _step("call_head64", path="call", hkv=8, d=64, logits="f32", s_lo=3000, s_hi=3000, n_lo=48, n_hi=48, vocab=128256),
        # fp32 throughout, head_dim 128: runs made to compare implementations
        _step("f32_1500", hq=16, hkv=8, dtype="f32", logits="f32", s_lo=1500, s_hi=1500, n_lo=40, n_hi=40),
        # grouped queries, many nodes
        _step("gqa_8k", hkv=8, s_lo=8192, s_hi=8192, n_lo=128, n_hi=128, depth=8, accept=0.5),
        # a serving batch of short grouped-query requests; a vocabulary whose rows are not 16-byte aligned
        _step("gqa_batch", hkv=8, batch=8, s_lo=100, s_hi=2000, n_lo=16, n_hi=48, depth=8, vocab=33333, shape_seed=3),
        # a serving batch over a paged cache, lengths spread widely
        _step("ragged_paged", batch=16, s_lo=512, s_hi=16384, n_lo=32, n_hi=96, depth=8, block=16, shape_seed=4),
        # every layer of a model: attention in each, one verification, one compaction
        _step("model_32", path="model", layers=32),
        # the largest: a long document, the largest tree
        _step("long_64k", hq=40, hkv=40, s_lo=65536, s_hi=65536, n_lo=256, n_hi=256, depth=10, vocab=128256, accept=0.4),
        # the drafter's side of a request: tables set up, prompt taken in, trees grown and the table updated
        dict(name="draft_request", path="draft", prompt=2048, steps=64, budget=64, depth=6, ll=2, fl=3, lc=8192, fc=4, vocab=32000, frozen=0),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    if rng.random() < 0.08:
        return dict(path="draft", prompt=_log(rng, 256, 16384), steps=_log(rng, 8, 128), budget=rng.choice([16, 64, 96, 128]),
                    depth=rng.randint(4, 10), ll=rng.randint(1, 2), fl=3, lc=8192, fc=rng.choice([4, 8, 16]), vocab=32000,
                    frozen=rng.choice([0, 0, 20000]))
    kind = rng.choices(["mfma", "head64", "f32"], [0.76, 0.12, 0.12])[0]
    c = dict(_STEP, path=rng.choices(["device", "host", "call", "model"], [0.5, 0.25, 0.1, 0.15])[0])
    c["depth"], c["accept"], c["shape_seed"] = rng.randint(4, 10), rng.choice([0.4, 0.5, 0.6]), rng.randrange(1000)
    c["vocab"] = rng.choice([1000, 32000, 32000, 33333, 128256])
    c["head_major"] = rng.random() < 0.15
    if kind == "mfma":
        c["hq"], c["hkv"] = rng.choice([(8, 8), (32, 32), (32, 32), (32, 8), (32, 8), (40, 40)])
        c["logits"] = rng.choice(["bf16", "bf16", "f32"])
        c["batch"] = 1 if rng.random() < 0.6 else _log(rng, 2, 32)
        c["block"] = rng.choice([0, 0, 16])
        s_hi = _log(rng, 16, 65536)
        n_hi = _log(rng, 1, 256)
    elif kind == "head64":
        c["hq"], c["hkv"], c["d"] = rng.choice([(32, 8, 64), (8, 8, 64)])
        c["logits"] = rng.choice(["bf16", "f32"])
        c["batch"] = rng.choice([1, 1, 2, 4])
        s_hi = _log(rng, 16, 4096)
        n_hi = _log(rng, 1, 64)
    else:
        c["hq"], c["hkv"], c["d"] = rng.choice([(8, 8, 64), (8, 8, 128), (16, 8, 128)])
        c["dtype"] = c["logits"] = "f32"
        s_hi = _log(rng, 16, 2048)
        n_hi = _log(rng, 1, 64)
    eb = 4 if c["dtype"] == "f32" else 2
    c["layers"] = rng.choice([2, 8, 32]) if c["path"] == "model" else 1
    # no more K/V, arithmetic and logits than the largest listed cases
    while c["layers"] * c["batch"] * (s_hi + n_hi) * c["hkv"] * c["d"] * 2 * eb > 1.2e9 or \
            4.0 * c["layers"] * c["batch"] * n_hi * c["hq"] * s_hi * c["d"] > 3.0e11 or c["batch"] * n_hi * c["vocab"] * 4 > 3e8:
        if c["batch"] > 1:
            c["batch"] //= 2
        elif c["layers"] > 1:
            c["layers"] //= 2
        else:
            s_hi = s_hi * 3 // 4
            n_hi = max(1, n_hi * 3 // 4)
    c["s_hi"], c["n_hi"] = s_hi, n_hi
    c["s_lo"] = s_hi if c["batch"] == 1 else max(1, s_hi // rng.choice([1, 4, 32]))
    c["n_lo"] = n_hi if c["batch"] == 1 else max(1, n_hi // rng.choice([1, 3]))
    return c


def _shapes(case):
    """(prefix lengths, tree sizes) of the case's sequences; the first one is as long as the range allows."""
    r = random.Random(1000 + case["shape_seed"])
    s = [case["s_hi"]] + [r.randint(case["s_lo"], case["s_hi"]) for _ in range(case["batch"] - 1)]
    n = [case["n_hi"]] + [r.randint(case["n_lo"], case["n_hi"]) for _ in range(case["batch"] - 1)]
    return s, n


def _prepare_step(case, seed):
    rng = np.random.default_rng(seed)
    gen = torch.Generator(device="cuda").manual_seed(seed)
    s, n = _shapes(case)
    batch, d, hkv, nl, V = case["batch"], case["d"], case["hkv"], case["layers"], case["vocab"]
    dt = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    lt = torch.float32 if case["logits"] == "f32" else torch.bfloat16
    total = sum(n)
    randn = lambda *shape, dtype=dt: torch.randn(*shape, generator=gen, device="cuda", dtype=dtype)  # noqa: E731

    # queries a little longer than the keys' scale: scores of standard deviation 1.5
    q = randn(nl, total, case["hq"], d) * 1.5
    table = None
    if case["block"]:
        need = [-(-(a + b) // case["block"]) for a, b in zip(s, n)]
        perm = rng.permutation(sum(need)).astype(np.int32)
        ids = np.full((batch, max(need)), -1, dtype=np.int32)
        at = 0
        for b, nb in enumerate(need):
            ids[b, :nb] = perm[at:at + nb]
            at += nb
        table = torch.from_numpy(ids).cuda()
        rows, per = sum(need), case["block"]
    else:
        rows, per = batch, max(a + b for a, b in zip(s, n))
    shape = (rows, hkv, per, d) if case["head_major"] else (rows, per, hkv, d)
    k, v = randn(nl, *shape), randn(nl, *shape)
    logits = randn(total, V, dtype=lt)

    # trees of random shape and tokens; at a node, with probability `accept`, the model generates what one of
    # its children drafted
    parents, tokens, planted = [], [], []
    for b in range(batch):
        par, _ = W.random_tree(rng, n[b], 4, case["depth"], False)
        tok = rng.integers(0, V, size=n[b]).astype(np.int32)
        kids = [[] for _ in par]
        for i in range(1, n[b]):
            kids[par[i]].append(i)
        base = sum(n[:b])
        for i, ks in enumerate(kids):
            if ks and rng.random() < case["accept"]:
                planted.append((base + i, int(tok[ks[int(rng.integers(len(ks)))]])))
        parents.append(par)
        tokens.append(tok)
    if planted:
        at = torch.tensor(planted, device="cuda")
        logits[at[:, 0], at[:, 1]] = 8.0
    parent, token = np.concatenate(parents).astype(np.int32), np.concatenate(tokens).astype(np.int32)
    kv_len = np.asarray(s, dtype=np.int32)
    offsets = np.concatenate([[0], np.cumsum(n)]).astype(np.int32)

    cfg = B.make_config(case["hq"], hkv, d, case["dtype"], case["logits"], batch, max(n), case["depth"], V, case["block"])
    ver = B.Verifier(cfg)
    layout = B.CB_LAYOUT_HEAD_MAJOR if case["head_major"] else B.CB_LAYOUT_TOKEN_MAJOR
    kvs = [B.kv_layer(k[i], v[i], table, layout, paged=case["block"] > 0) for i in range(nl)]
    out = torch.zeros_like(q)
    st = dict(case=case, ver=ver, k=k, v=v, out=out, q=q, logits=logits, table=table, kvs=kvs)
    if case["path"] == "host":
        hs = ver.bind_host_step(q[0], kvs[0], logits, out[0], batch=batch, layers=kvs)
        hs.kv_len[:], hs.node_offsets[:] = kv_len, offsets
        hs.parent[:total], hs.tokens[:total] = parent, token
        st.update(step=hs)
    elif case["path"] == "call":
        st.update(args=(q[0], kvs[0], kv_len, offsets, parent, token, logits, out[0]))
    else:
        d_len = torch.zeros(batch, dtype=torch.int32, device="cuda")
        d_tok = torch.zeros(batch, case["depth"] + 1, dtype=torch.int32, device="cuda")
        d_par, d_tk = torch.from_numpy(parent).cuda(), torch.from_numpy(token).cuda()
        if case["path"] == "model":
            step = ver.bind_model_step(list(q), kvs, kv_len, offsets, d_par, d_tk, logits, list(out), d_len, d_tok)
        else:
            step = ver.bind_step(q[0], kvs[0], kv_len, offsets, d_par, d_tk, logits, out[0], d_len, d_tok, kvs)
        st.update(step=step, len=d_len, tok=d_tok, tree=(d_par, d_tk))
    return st


def _prepare_draft(case, seed):
    rng = np.random.default_rng(seed)
    text = W.zipf_stream(rng, case["prompt"] + 3 * case["steps"] + case["fl"], case["vocab"])
    corpus = W.zipf_stream(rng, case["frozen"], case["vocab"]) if case["frozen"] else None
    return dict(case=case, text=np.ascontiguousarray(text, dtype=np.int32), corpus=corpus)


def prepare(case, seed):
    return _prepare_draft(case, seed) if case["path"] == "draft" else _prepare_step(case, seed)


def _run_draft(state):
    """A request's drafting: fresh tables, the prompt, then a tree and an update for every step (of 1 to 3
    tokens, as acceptance would have it)."""
    c, text = state["case"], state["text"]
    table = B.DraftTable(c["ll"], c["fl"], c["lc"], c["fc"])
    tables = [table]
    if state["corpus"] is not None:
        tables.append(B.DraftTable(c["ll"], c["fl"], c["lc"], c["fc"], frozen_from=state["corpus"]))
    grower = B.TreeGrower(tables, c["budget"], c["depth"])
    n = c["prompt"]
    table.update(text[:n], 0)
    trees = np.full((3, c["steps"], c["budget"]), -1, dtype=np.int32)
    for i in range(c["steps"]):
        parent, token, depth = grower.grow(text, n)
        trees[0, i, :len(parent)], trees[1, i, :len(parent)], trees[2, i, :len(parent)] = parent, token, depth
        old, n = n, n + 1 + i % 3
        table.update(text[:n], old - (c["fl"] - 1))
    size = table.size()
    for t in tables:
        t.close()
    return dict(trees=trees, leaders=size[0], followers=size[1])


def run(state):
    path = state["case"]["path"]
    if path == "draft":
        return _run_draft(state)
    out = dict(attention=state["out"], k=state["k"], v=state["v"])
    if path == "host":
        step = state["step"]
        step.verify()
        step.compact()
        out.update(accepted_len=step.accepted_len, accepted_tokens=step.accepted_tokens)
    elif path == "call":
        _, acc_len, acc_tok = state["ver"].verify_tree(*state["args"])
        new_len = state["ver"].compact_kv(state["kvs"], state["case"]["batch"])
        out.update(accepted_len=acc_len, accepted_tokens=acc_tok, new_len=new_len)
    else:
        state["step"]()
        out.update(accepted_len=state["len"], accepted_tokens=state["tok"])
    return out


def work(case):
    if case["path"] == "draft":
        tokens = case["prompt"] + 2 * case["steps"] + case["frozen"]
        # every window's leader and follower hashed and stored once, every tree written once
        return {"bytes": tokens * (case["ll"] + case["fl"]) * 4 + 3 * case["steps"] * case["budget"] * 4, "flops": 0}
    s, n = _shapes(case)
    eb, lb = (4 if case["dtype"] == "f32" else 2), (4 if case["logits"] == "f32" else 2)
    slots, nodes = sum(s) + sum(n), sum(n)
    attention = slots * case["hkv"] * case["d"] * 2 * eb + nodes * case["hq"] * case["d"] * 2 * eb
    tree = nodes * 8 + case["batch"] * (case["depth"] + 2) * 4
    moved = case["batch"] * case["hkv"] * case["d"] * 2 * eb * 2        # one accepted node, read and written
    flops = sum(4.0 * b * case["hq"] * case["d"] * (a + min(b, case["depth"])) for a, b in zip(s, n))
    return {"bytes": case["layers"] * (attention + moved) + tree + nodes * case["vocab"] * lb, "flops": case["layers"] * flops}


def tolerance(case):
    if case["path"] == "draft":
        return "exact"
    # attention: bf16 results of fp32 sums with bf16 probabilities and partial sums; fp32 otherwise.  Tokens,
    # lengths and cache contents are exact (whole numbers may not differ; the caches are copies).
    return {"rel": 1e-5, "max": 1e-4} if case["dtype"] == "f32" else {"rel": 1e-2, "max": 5e-2}
