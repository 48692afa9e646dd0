"""A verification and its compaction as one call (cb_verify_and_compact_device, what bind_step makes) against the two calls: the same
attention, acceptance and cache bytes, step after step, whichever of a head's attention and the acceptance is through first."""
import numpy as np
import pytest

from paper_2511_21699_amd import binding as B
from paper_2511_21699_amd import workloads as W
from .gpu_harness import accept_to_the_last_node, step_info

pytestmark = pytest.mark.gpu

CASES = [  # dtype, heads, kv heads, head_dim, vocabulary, prefixes, tree sizes, options, paged
    ("bf16", 8, 8, 128, 1000, [1500], [40], {}, False),
    ("bf16", 8, 8, 128, 128256, [0], [64], {}, False),                    # the acceptance is last
    ("bf16", 32, 8, 128, 90000, [5], [16], {}, True),
    ("bf16", 4, 4, 128, 500, [100], [256], {"splits": 11}, False),        # the tree in 9 splits
    ("bf16", 4, 4, 128, 500, [95], [64], {"splits": 5}, True),            # and in 3, several at its edge
    ("bf16", 32, 4, 128, 3000, [700, 64, 31], [130, 256, 1], {}, False),  # several row tiles
    ("bf16", 32, 8, 128, 60000, [40, 2000], [20, 3], {"fuse_logits": 0}, True),
    ("bf16", 16, 8, 128, 2000, [900] * 5, [50] * 5, {"external_merge": 1, "splits": 3}, False),
    ("bf16", 16, 8, 128, 2000, [900] * 5, [50] * 5, {"coop_merge": 0, "splits": 3}, False),
    ("bf16", 8, 2, 64, 700, [300, 10], [64, 33], {}, True),
    ("bf16", 32, 8, 64, 33333, [1200], [100], {"splits": 4}, False),
    ("f32", 8, 8, 64, 1000, [256], [15], {}, False),
    ("f32", 16, 8, 128, 50000, [33, 700], [40, 17], {}, True),
    ("f32", 6, 3, 128, 300, [120], [64], {"splits": 5}, False),
    ("bf16", 8, 8, 128, 1000, [600], [40], {"attn_impl": 1}, False),      # (the scalar kernels: two launches)
    ("bf16", 32, 8, 128, 3000, [500], [100], {"tile_rows": 64}, False),   # 7 tiles of 64 rows that a head's move waits for
    ("bf16", 32, 8, 128, 3000, [500], [100], {"tile_rows": 128}, True),   # 4 of 128
    ("bf16", 4, 4, 128, 500, [300, 31], [256, 70], {"tile_rows": 64}, True),
    ("bf16", 8, 2, 64, 700, [900], [90], {"tile_rows": 128}, False),
    ("bf16", 40, 40, 128, 32000, [790], [97], {"tile_rows": 256}, False), # 10 heads to a wave of the acceptance's workgroup, 4 at a time
    ("bf16", 44, 22, 128, 20000, [300, 20], [70, 40], {"tile_rows": 128}, True),
]
TWO_LAUNCHES = {"attn_impl", "many"}
for n in (16, 17, 40):  # sequences that 8 logits workgroups accept, two each and more; these with head_dim 64 in bf16 have a launch for their compaction
    lens, sizes, many = [5 + 7 * i % 90 for i in range(n)], [3 + i % 6 for i in range(n)], {"logits_wgs": 8}
    CASES += [("bf16", 8, 8, 128, 300, lens, sizes, many, False), ("f32", 4, 4, 64, 300, lens, sizes, many, False),
              ("f32", 8, 4, 128, 300, lens, sizes, many, n == 16), ("bf16", 8, 4, 64, 300, lens, sizes, dict(many, many=1) if n > 16 else many, False)]
CASES += [("bf16", 16, 8, 128, 300, [40 * i for i in range(n)], [9 + i for i in range(n)], {"logits_wgs": 8}, False) for n in (9, 12)]
CASES += [("bf16", 72, 72, 64, 300, [20 * i for i in range(8)], [9 + i for i in range(8)], {"logits_wgs": 8}, False)]   # more heads than lanes


@pytest.mark.parametrize("i", range(len(CASES)))
@pytest.mark.parametrize("layout", [B.CB_LAYOUT_TOKEN_MAJOR, B.CB_LAYOUT_HEAD_MAJOR])
def test_one_call_against_two(i, layout):
    import torch
    dtype, hq, hkv, d, vocab, lens, nodes, options, paged = CASES[i]
    print(f"[case] step {CASES[i]} layout={layout}", flush=True)
    rng = np.random.default_rng(i)
    pars = [W.random_tree(rng, n, 2, 13, False)[0] for n in nodes]
    case = W.custom_case(7000 + i, dtype, len(lens), hq, hkv, d, vocab, lens, pars, paged=paged, p_match=0.95)
    total, moved = case.total_nodes, 0
    got = []
    for fused in (True, False):
        dc = B.DeviceCase(case, layout=layout)
        ver = B.Verifier(B.config_for_case(case))
        for k, v in options.items():
            if k != "many":
                ver.set_option(k, v)
        par, tok = torch.from_numpy(case.parent).cuda(), torch.from_numpy(case.tokens).cuda()
        out, k0 = torch.zeros_like(dc.q), dc.k.clone()
        n, t = torch.zeros(len(lens), dtype=torch.int32, device="cuda"), torch.zeros(len(lens), case.max_depth + 1, dtype=torch.int32, device="cuda")
        step = ver.bind_step(dc.q, dc.kv, case.kv_len, case.node_offsets, par, tok, dc.logits, out, n, t, [dc.kv])
        for _ in range(3):
            if fused:
                step()
                info = step_info(ver)
                assert info["moved"] == (not TWO_LAUNCHES & set(options) and (len(lens) == 1 or not paged)) and info["tile_rows"] == options.get("tile_rows", info["tile_rows"])
            else:
                ver.verify_tree_device(dc.q, dc.kv, case.kv_len, case.node_offsets, par, tok, dc.logits, out, n, t)
                ver.compact_kv([dc.kv], len(lens), want_len=False)
            torch.cuda.synchronize()
            got.append((out.clone(), dc.k.clone(), dc.v.clone(), n.clone(), t.clone(), ver.get_path(len(lens)), ver.get_argmax(total)))
        moved += int(not torch.equal(dc.k, k0))
        ver.close()
    for rep in range(3):
        for a, b in zip(got[rep], got[3 + rep]):
            assert (torch.equal(a, b) if isinstance(a, torch.Tensor) else np.array_equal(a, b)), f"step {rep}"
    assert moved in (0, 2) and (moved == 2 or max(int(x) for x in got[0][3]) < 3)


def test_operands_that_overlap_the_cache_take_two_launches():
    """Queries that lie in the cache's memory: rows that move must not reach them before they are read."""
    import torch
    case = W.custom_case(7100, "bf16", 1, 8, 8, 128, 500, [300], [W.random_tree(np.random.default_rng(1), 40, 2, 9, False)[0]], p_match=0.95)
    ref = None
    for inside in (False, True):
        dc = B.DeviceCase(case)
        q = dc.k[0, 300:340] if inside else dc.k[0, 300:340].clone()   # ([nodes][heads][D], as the queries are)
        ver = B.Verifier(B.config_for_case(case))
        par, tok = torch.from_numpy(case.parent).cuda(), torch.from_numpy(case.tokens).cuda()
        out = torch.zeros_like(dc.q)
        n, t = torch.zeros(1, dtype=torch.int32, device="cuda"), torch.zeros(1, case.max_depth + 1, dtype=torch.int32, device="cuda")
        ver.bind_step(q, dc.kv, case.kv_len, case.node_offsets, par, tok, dc.logits, out, n, t, [dc.kv])()
        torch.cuda.synchronize()
        ref = ref or (out, dc.k.clone())
        assert torch.equal(out, ref[0]) and torch.equal(dc.k, ref[1])
        ver.close()


@pytest.mark.parametrize("layers", [1, 2])
def test_operands_in_a_cache_of_any_size(layers):
    """A descriptor's capacity may be just a large number (of one sequence only the length is looked at); 2^53 slots of 2 KiB are 2^64 bytes."""
    import torch
    case = W.custom_case(7150, "bf16", 1, 8, 8, 128, 500, [300], [W.random_tree(np.random.default_rng(1), 40, 2, 9, False)[0]], p_match=0.95, extra_capacity=100)
    for capacity in (None, 2 ** 53):
        dc = B.DeviceCase(case)
        dc.kv.capacity_or_num_blocks = capacity or dc.kv.capacity_or_num_blocks
        q, outs = dc.k[0, 300:340], [dc.k[0, 380:420], torch.zeros_like(dc.q)]   # ([nodes][heads][D], as the queries are)
        ver = B.Verifier(B.config_for_case(case))
        par, tok = torch.from_numpy(case.parent).cuda(), torch.from_numpy(case.tokens).cuda()
        n, t = torch.zeros(1, dtype=torch.int32, device="cuda"), torch.zeros(1, case.max_depth + 1, dtype=torch.int32, device="cuda")
        if layers == 1:
            ver.bind_step(q, dc.kv, case.kv_len, case.node_offsets, par, tok, dc.logits, outs[1], n, t, [dc.kv])()
        else:
            ver.bind_model_step([q, q], [dc.kv, dc.kv], case.kv_len, case.node_offsets, par, tok, dc.logits, outs, n, t)()
        torch.cuda.synchronize()
        info = step_info(ver)
        assert not info["moved"] and not info["layers"], (capacity, info)
        ver.close()


def test_a_sequence_that_is_in_a_paged_batch_twice():
    """Rows of the block table that share the blocks with the tree: no row moves while the other sequence reads it."""
    import torch
    tree, n = [-1, 0, 0] + [1] * 37, 40                                      # accepted: 0, 2
    case = W.custom_case(7160, "bf16", 2, 8, 8, 128, 500, [300, 300], [tree, tree], paged=True, p_match=0.0)
    case.block_table[1] = case.block_table[0]
    for x in (case.q, case.logits):
        x[n:] = x[:n]
    arg = np.argmax(W.to_f64(case.logits, case.dtype), axis=1)
    case.tokens = np.asarray([(arg[p] + 1) % 500 for p in case.parent], dtype=np.int32)
    case.tokens[2] = case.tokens[n + 2] = arg[0]
    got = []
    for fused in (True, False):
        dc, ver = B.DeviceCase(case), B.Verifier(B.config_for_case(case))
        par, tok, out = torch.from_numpy(case.parent).cuda(), torch.from_numpy(case.tokens).cuda(), torch.zeros_like(dc.q)
        m, t = torch.zeros(2, dtype=torch.int32, device="cuda"), torch.zeros(2, case.max_depth + 1, dtype=torch.int32, device="cuda")
        if fused:
            ver.bind_step(dc.q, dc.kv, case.kv_len, case.node_offsets, par, tok, dc.logits, out, m, t, [dc.kv])()
            assert not step_info(ver)["moved"]
        else:
            ver.verify_tree_device(dc.q, dc.kv, case.kv_len, case.node_offsets, par, tok, dc.logits, out, m, t)
            ver.compact_kv([dc.kv], 2, want_len=False)
        torch.cuda.synchronize()
        assert m.tolist() == [1, 1] and torch.equal(out[:n], out[n:])
        got.append((out, dc.k, dc.v, t))
        ver.close()
    assert all(torch.equal(a, b) for a, b in zip(*got))


def chain(n):
    """A path of n - 2 nodes below the root, each a slot away from its place: node 1 is a leaf beside it."""
    return [-1, 0, 0] + list(range(2, n - 1))


@pytest.mark.parametrize("dtype,hq,hkv,d", [("bf16", 4, 4, 128), ("bf16", 16, 8, 64), ("f32", 4, 2, 128), ("f32", 8, 8, 64)])
@pytest.mark.parametrize("sizes", [[65], [66], [67], [130], [256], [200, 3, 70]])   # accepted: 63, 64, 65, 128, 254 nodes
@pytest.mark.parametrize("paged", [False, True])
def test_paths_longer_than_a_wave(dtype, hq, hkv, d, sizes, paged):
    """Paths of more nodes than a wavefront has lanes, all of which move, against the oracle's cache."""
    import torch
    from oracle import cb_oracle as O
    print(f"[case] long paths {dtype} {hq}/{hkv} x {d} {sizes} paged={paged}", flush=True)
    case = W.custom_case(7200 + sum(sizes), dtype, len(sizes), hq, hkv, d, 300, [50 + 9 * b for b in range(len(sizes))], [chain(n) for n in sizes],
                         paged=paged, p_match=0.0)
    res = accept_to_the_last_node(case)
    dc = B.DeviceCase(case)
    ver = B.Verifier(B.config_for_case(case))
    par, tok = torch.from_numpy(case.parent).cuda(), torch.from_numpy(case.tokens).cuda()
    n, t = torch.zeros(case.B, dtype=torch.int32, device="cuda"), torch.zeros(case.B, case.max_depth + 1, dtype=torch.int32, device="cuda")
    ver.bind_step(dc.q, dc.kv, case.kv_len, case.node_offsets, par, tok, dc.logits, torch.zeros_like(dc.q), n, t, [dc.kv])()
    torch.cuda.synchronize()
    assert step_info(ver)["moved"] == (not paged or case.B == 1)
    k, v = case.k.copy(), case.v.copy()
    for b, (L, path, _) in enumerate(res):
        assert int(n[b]) == L == sizes[b] - 2
        O.compact(case, k, v, b, path)
    assert np.array_equal(B.to_host(dc.k, dtype), k) and np.array_equal(B.to_host(dc.v, dtype), v)
    ver.close()
