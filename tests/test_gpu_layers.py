"""A model's step as one call (cb_model_step_device): layers that are attended to in one launch against the oracle, and the calls whose
layers have to go one by one."""
import copy

import numpy as np
import pytest

from paper_2511_21699_amd import binding as B
from paper_2511_21699_amd import workloads as W
from .gpu_harness import check_attention, step_info, structured_rows

pytestmark = pytest.mark.gpu

CASES = [  # dtype, heads, kv heads, head_dim, vocabulary, prefixes, tree sizes, layers, paged, layout, launches
    ("bf16", 8, 8, 128, 1000, [200], [40], 5, False, 0, 1),
    ("bf16", 32, 32, 128, 90000, [0], [1], 32, False, 0, 1),              # 1024 tiles of one key
    ("bf16", 8, 8, 128, 700, [60], [64], 33, True, 0, 1),                 # one more than a launch serves
    ("bf16", 8, 8, 128, 3000, [3000], [33], 2, False, 1, 1),              # splits, merged cooperatively
    ("bf16", 32, 32, 128, 3000, [3000], [20], 3, True, 0, 1),             # and by the last to arrive
    ("bf16", 16, 8, 128, 700, [300, 31, 0], [17, 32, 5], 4, True, 0, 1),  # a batch, longest first
    ("bf16", 6, 3, 128, 700, [257, 64], [9, 30], 3, False, 0, 1),         # kv heads no multiple of 8
    ("bf16", 32, 8, 128, 700, [400], [70], 4, True, 0, 1),                # wide tiles, two to a head
    ("bf16", 16, 2, 128, 700, [900, 100], [33, 12], 3, False, 1, 1),
    ("bf16", 8, 2, 64, 700, [1500], [12], 3, False, 0, 1),                # head_dim 64
    ("bf16", 16, 8, 64, 700, [130, 700], [64, 40], 3, True, 0, 1),
    ("f32", 8, 8, 64, 1000, [256], [15], 6, False, 0, 1),
    ("f32", 4, 2, 128, 300, [900, 20], [64, 7], 3, True, 0, 1),           # splits
]


def step_of(case, layers, layout):
    import torch
    cases = [case]
    for i in range(1, layers):
        c = copy.copy(case)
        rng = np.random.default_rng(900 + i)
        perm = rng.permutation(case.Hq)
        c.q = np.ascontiguousarray(case.q[:, perm])                       # other queries, keys and values of the same kinds
        c.k, c.v = np.ascontiguousarray(np.roll(case.k, i, axis=-1)), np.ascontiguousarray(np.roll(case.v, 3 * i, axis=-1))
        cases.append(c)
    dcs = [B.DeviceCase(c, layout=layout) for c in cases]
    kvs = [B.kv_layer(dc.k, dc.v, dcs[0].block_table, layout, paged=case.block_size > 0) for dc in dcs]
    par, tok = torch.from_numpy(case.parent).cuda(), torch.from_numpy(case.tokens).cuda()
    n = torch.zeros(case.B, dtype=torch.int32, device="cuda")
    t = torch.zeros(case.B, case.max_depth + 1, dtype=torch.int32, device="cuda")
    return cases, dcs, kvs, par, tok, n, t


def check_caches(cases, dcs, res, layout):
    from oracle import cb_oracle as O
    for c, dc in zip(cases, dcs):
        k, v = c.k.copy(), c.v.copy()
        for b, (_, path, _) in enumerate(res):
            O.compact(c, k, v, b, path)
        got = [B.to_host(x, c.dtype) for x in (dc.k, dc.v)]
        if layout == B.CB_LAYOUT_HEAD_MAJOR:
            got = [x.swapaxes(1, 2) for x in got]
        assert np.array_equal(got[0], k) and np.array_equal(got[1], v)


@pytest.mark.parametrize("i", range(len(CASES)))
def test_layers_in_one_launch(i):
    import torch
    from oracle import cb_oracle as O
    dtype, hq, hkv, d, vocab, lens, nodes, layers, paged, layout, kernels = CASES[i]
    print(f"[case] layers {CASES[i]}", flush=True)
    rng = np.random.default_rng(i)
    pars = [W.random_tree(rng, n, 2, 9, False)[0] for n in nodes]
    case = W.custom_case(8000 + i, dtype, len(lens), hq, hkv, d, vocab, lens, pars, paged=paged, p_match=0.9)
    cases, dcs, kvs, par, tok, n, t = step_of(case, layers, layout)
    ver = B.Verifier(B.config_for_case(case))
    outs = [torch.zeros_like(dc.q) for dc in dcs]
    step = ver.bind_model_step([dc.q for dc in dcs], kvs, case.kv_len, case.node_offsets, par, tok, dcs[-1].logits, outs, n, t)
    k0 = [(dc.k.clone(), dc.v.clone()) for dc in dcs]
    first = None
    _, res = O.verify(case)
    for _ in range(3):                                                     # (counters are left as they were found)
        for dc, (k, v) in zip(dcs, k0):
            dc.k.copy_(k)
            dc.v.copy_(v)
        step()
        torch.cuda.synchronize()
        first = first or [o.clone() for o in outs]
        assert all(torch.equal(a, b) for a, b in zip(first, outs))
        assert n.cpu().tolist() == [r[0] for r in res]
        for b, (L, _, toks) in enumerate(res):
            assert t[b, :L + 1].cpu().tolist() == toks.tolist()
        check_caches(cases, dcs, res, layout)
    assert ver.device_status() & 3 == 0 and ver.last_launch_info()["kernels"] == kernels
    info = step_info(ver)
    assert info["layers"] == layers and info["launches"] == -(-layers // 32), info
    rows = structured_rows(case)
    for c, out in zip(cases, outs):
        got = W.to_f64(B.to_host(out, dtype), dtype)
        check_attention(case, np.stack([got[case.node_offsets[b] + x, h] for b, h, x in rows]), O.attention_rows(c, rows), "layer")
    ver.close()


@pytest.mark.parametrize("kind", ["chained", "one output", "splits", "tile rows"])
def test_layers_that_go_one_by_one(kind):
    """A layer's result as the next one's queries, or all in one place: the layers follow each other; options too."""
    import torch
    rng = np.random.default_rng(3)
    case = W.custom_case(8100, "bf16", 1, 8 if kind != "tile rows" else 32, 8, 128, 500, [300], [W.random_tree(rng, 40, 2, 9, False)[0]], p_match=0.95)
    got = []
    for together in (True, False):
        _, dcs, kvs, par, tok, n, t = step_of(case, 3, 0)
        outs = [torch.zeros_like(dc.q) for dc in dcs]
        qs = [dc.q for dc in dcs]
        ver = B.Verifier(B.config_for_case(case))
        if kind == "chained":
            qs = [qs[0], outs[0], outs[1]]
        elif kind == "one output":
            outs = [outs[0]] * 3
        elif kind == "splits":
            ver.set_option("splits", 3)
        else:
            ver.set_option("tile_rows", 128)
        if together:
            ver.bind_model_step(qs, kvs, case.kv_len, case.node_offsets, par, tok, dcs[-1].logits, outs, n, t)()
        else:
            for q, kv, out in zip(qs[:2], kvs, outs):
                ver.tree_attention_device(q, kv, case.kv_len, case.node_offsets, par, out)
            ver.verify_tree_device(qs[2], kvs[2], case.kv_len, case.node_offsets, par, tok, dcs[-1].logits, outs[2], n, t)
            ver.compact_kv(kvs, 1, want_len=False)
        torch.cuda.synchronize()
        assert step_info(ver)["layers"] == 0 and step_info(ver)["tile_rows"] == (64 if kind != "tile rows" else 128)
        got.append([x.clone() for x in outs] + [dc.k.clone() for dc in dcs] + [n.clone(), t.clone()])
        ver.close()
    assert all(torch.equal(a, b) for a, b in zip(*got))
