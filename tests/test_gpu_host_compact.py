"""Compaction behind the host-array form, which leaves the launch out where the accepted paths are the trees' first nodes: cache bytes and
lengths against the oracle, with paths that move and paths that do not, alone and side by side."""
import numpy as np
import pytest

from oracle import cb_oracle as O
from paper_2511_21699_amd import binding as B
from paper_2511_21699_amd import workloads as W

pytestmark = pytest.mark.gpu

CHAIN = [-1, 0, 1, 2, 3, 4]                      # whatever is accepted is in place
LATE = [-1, 0, 0, 2, 2, 4]                       # accepted: 2, 4, 5
FORK = [-1, 0, 1, 1, 3, 4]                       # 1 in place, then 3, 4, 5
WIDE = [-1] + [0] * 70 + [70, 71, 72]            # more than 64 nodes: 70 .. 73
LONG = list(range(-1, 70))                       # more than 64 nodes, in place
ROOT = [-1]


@pytest.mark.parametrize("full_sync", [0, 1])
@pytest.mark.parametrize("trees", [[CHAIN], [LATE], [FORK], [WIDE], [LONG], [ROOT], [CHAIN, LATE], [FORK, CHAIN, ROOT], [CHAIN, LONG], [ROOT, ROOT]])
def test_compaction_behind_the_host_form(trees, full_sync):
    import torch
    print(f"[case] {[len(t) for t in trees]} full_sync={full_sync}", flush=True)
    case = W.custom_case(8300 + len(trees), "bf16", len(trees), 4, 4, 128, 500, [40 + 7 * b for b in range(len(trees))], trees, p_match=0.0)
    # tokens: every node on the way to the last one matches its parent's row, no other does
    arg = O.argmax(case.logits, case.dtype)
    tokens = np.where(arg == 0, 1, 0).astype(np.int32)
    for b, par in enumerate(trees):
        lo, x = int(case.node_offsets[b]), len(par) - 1
        for i in range(1, len(par)):
            tokens[lo + i] = (arg[lo + par[i]] + 1) % 500
        while x > 0:
            tokens[lo + x] = arg[lo + par[x]]
            x = par[x]
    case.tokens = tokens
    _, res = O.verify(case)
    assert [int(r[1][r[0]]) for r in res] == [len(t) - 1 for t in trees]
    dc = B.DeviceCase(case)
    ver = B.Verifier(B.config_for_case(case))
    ver.set_option("full_sync", full_sync)
    _, acc_len, _ = ver.verify_tree(dc.q, dc.kv, case.kv_len, case.node_offsets, case.parent, case.tokens, dc.logits)
    new_len = ver.compact_kv([dc.kv], case.B)
    torch.cuda.synchronize()
    k, v = case.k.copy(), case.v.copy()
    for b, (L, path, _) in enumerate(res):
        assert acc_len[b] == L and O.compact(case, k, v, b, path) == new_len[b]
    assert np.array_equal(B.to_host(dc.k, case.dtype), k) and np.array_equal(B.to_host(dc.v, case.dtype), v)
    ver.close()
