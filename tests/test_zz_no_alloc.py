"""cb_tree_attention_noalloc (the entry point for callers that cannot allocate) against
cb_tree_attention_device on the same inputs: the same kernels run with the scratch memory taken from
the library's fixed device array instead of a caller's workspace, so the outputs must be identical
bit for bit, and within the attention tolerance of the oracle.  Two calls in a row, the second with
a smaller input, share the array."""
import numpy as np
import pytest

from paper_2511_21699_amd import binding as B
from paper_2511_21699_amd import workloads as W
from tests.gpu_harness import check_attention, sample_rows

pytestmark = pytest.mark.gpu


def _both(case, rows=None):
    import torch
    from oracle import cb_oracle as O
    dc = B.DeviceCase(case)
    cfg = B.config_for_case(case)
    d_par = torch.from_numpy(case.parent).cuda()
    ver = B.Verifier(cfg)
    ref = torch.zeros_like(dc.q)
    ver.tree_attention_device(dc.q, dc.kv, case.kv_len, case.node_offsets, d_par, ref)
    torch.cuda.synchronize()
    ver.close()
    out = torch.zeros_like(dc.q)
    B.tree_attention_noalloc(cfg, dc.q, dc.kv, case.kv_len, case.node_offsets, d_par, out)
    torch.cuda.synchronize()
    a, b = B.to_host(ref, case.dtype), B.to_host(out, case.dtype)
    assert np.array_equal(a, b), f"{case.name}: no-alloc entry point differs from cb_tree_attention_device"
    got = W.to_f64(b, case.dtype)
    if rows is None:
        check_attention(case, got, O.attention(case), case.name)
    else:
        sel = np.stack([got[case.node_offsets[bb] + i, h] for bb, h, i in rows])
        check_attention(case, sel, O.attention_rows(case, rows), case.name)


def test_no_alloc_entry_point_two_calls_in_a_row():
    big = W.make_config(2)                                  # 8 splits, cooperative merge, 4.3 MB of partials
    print("[case] no-alloc: 7B-shaped, full size", flush=True)
    _both(big, rows=sample_rows(big, 64, seed=5))
    rng = np.random.default_rng(77)
    small = W.custom_case(771, "bf16", 2, 8, 4, 128, 100, [700, 33], [W.random_tree(rng, 40, 3, 6, False)[0], W.chain_tree(9)], paged=True)
    print("[case] no-alloc: smaller paged batch right behind it", flush=True)
    _both(small)
    tiny = W.make_config(1)                                 # fp32: its own matrix-core kernel
    print("[case] no-alloc: tiny fp32", flush=True)
    _both(tiny)


def test_no_alloc_entry_point_with_fewer_splits_than_planned():
    """A call whose planned splits need more than the fixed array: fewer splits, the same tolerance."""
    import torch
    from oracle import cb_oracle as O
    rng = np.random.default_rng(78)
    nodes, lens = [128, 109, 107, 63], [1322, 542, 200, 290]
    case = W.custom_case(772, "bf16", 4, 64, 32, 128, 100, lens, [W.random_tree(rng, n, 4, 8, False)[0] for n in nodes], q_scale=2.0)
    print("[case] no-alloc: wide tiles beyond the scratch array at the planned splits", flush=True)
    dc = B.DeviceCase(case)
    out = torch.zeros_like(dc.q)
    B.tree_attention_noalloc(B.config_for_case(case), dc.q, dc.kv, case.kv_len, case.node_offsets, torch.from_numpy(case.parent).cuda(), out)
    torch.cuda.synchronize()
    got = W.to_f64(B.to_host(out, case.dtype), case.dtype)
    rows = sample_rows(case, 96, seed=6)
    check_attention(case, np.stack([got[case.node_offsets[b] + i, h] for b, h, i in rows]), O.attention_rows(case, rows), case.name)
