"""Verifications with wide tiles as one launch (logits workgroups in front of the attention's) and as two: the same
bytes either way, and the oracle's results."""
import numpy as np
import pytest

from paper_2511_21699_amd import binding as B
from paper_2511_21699_amd import workloads as W
from tests.gpu_harness import run_case, sample_rows

pytestmark = pytest.mark.gpu


# one tile and several, one sequence and several, one split and several, paged, logits that hide behind the sweep and
# logits that do not (a launch of their own)
@pytest.mark.parametrize("g,D,sizes,lens,V,dtype,paged,one", [
    (4, 128, [17], [700], 500, "bf16", False, True), (1, 128, [256], [3000], 1001, "bf16", False, True),
    (4, 64, [100], [900], 300, "bf16", True, True), (8, 128, [20, 3, 64], [900, 0, 2100], 777, "bf16", True, True),
    (4, 128, [64], [40], 9001, "bf16", False, False)])
def test_one_launch_and_two_agree(g, D, sizes, lens, V, dtype, paged, one):
    rng = np.random.default_rng(sum(sizes))
    pars = [W.random_tree(rng, n, 4, 7, False)[0] for n in sizes]
    case = W.custom_case(5600 + V, dtype, len(sizes), 2 * g, 2, D, V, lens, pars, paged=paged, q_scale=2.0, p_match=0.8)
    one_launch_and_two(case, one)


# Tiles of up to 128 rows in several rounds of workgroups (12 sequences x 32 heads on 256 compute units): two launches unless
# the sums are in 32 bits (head_dim 64; slices of the block table beyond 1022 entries) or a tile is larger.
@pytest.mark.parametrize("D,lens,block,first,one", [(128, range(400, 520, 10), 0, 70, False), (64, range(400, 520, 10), 0, 70, True),
                                                    (128, range(1100, 1220, 10), 1, 70, True), (128, range(400, 520, 10), 0, 129, True)])
def test_several_rounds(D, lens, block, first, one, monkeypatch):
    monkeypatch.setattr(W, "BLOCK_TOKENS", block)
    rng = np.random.default_rng(first)
    pars = [W.random_tree(rng, n, 4, 7, False)[0] for n in [first] + [70] * 11]
    case = W.custom_case(5700 + D, "bf16", 12, 32, 32, D, 300, list(lens), pars, paged=block > 0, q_scale=2.0, p_match=0.8)
    case.block_size = block
    one_launch_and_two(case, one)


def one_launch_and_two(case, one):
    import torch
    run_case(case, rows=sample_rows(case, 60), what=f"one launch {np.diff(case.node_offsets).tolist()}")
    dc = B.DeviceCase(case)
    got = []
    for fuse in (1, 0):
        ver = B.Verifier(B.config_for_case(case))
        ver.set_option("fuse_logits", fuse)
        out, acc_len, acc_tok = ver.verify_tree(dc.q, dc.kv, case.kv_len, case.node_offsets, case.parent, case.tokens, dc.logits)
        torch.cuda.synchronize()
        assert ver.last_launch_info()["fused"] == (fuse == 1 and one)
        got.append((B.to_host(out, "bf16").copy(), acc_len.copy(), acc_tok.copy(), ver.get_argmax(case.total_nodes), ver.get_path(case.B)))
        ver.close()
    for x, y in zip(got[0], got[1]):
        assert np.array_equal(x, y)
