"""Paged caches whose table slice of one split is longer than the part of it that the attention kernel keeps in
LDS at a time (1024 entries): the ring of table segments is refilled during the sweep."""
import numpy as np
import pytest

from paper_2511_21699_amd import binding as B
from paper_2511_21699_amd import workloads as W
from tests.gpu_harness import run_case, sample_rows

pytestmark = pytest.mark.gpu


# (block size, prefix, forced splits): a slice that just fits, one entry more, several refills at one token per
# block -- where the refills come closest to the requests -- and at 16
@pytest.mark.parametrize("block,S,splits", [(1, 960, 1), (1, 961, 1), (1, 3300, 1), (2, 5000, 2), (16, 16330, 1), (16, 33000, 1)])
@pytest.mark.parametrize("n", [33, 150])
def test_table_slices_beyond_the_lds_ring(block, S, splits, n, monkeypatch):
    monkeypatch.setattr(W, "BLOCK_TOKENS", block)
    par = W.random_tree(np.random.default_rng(S), n, 4, 7, False)[0]
    case = W.custom_case(4200 + S, "bf16", 1, 2, 2, 128, 500, [S], [par], paged=True, q_scale=2.0)
    case.block_size = block
    ver_rows = sample_rows(case, 60)
    run_case(case, rows=ver_rows, options={"splits": splits, "attn_impl": 2}, what=f"block {block} S={S}")


# The same at head_dim 64, whose 16 units in flight are 512 one-token entries -- two whole segments, as many as a refill may run
# ahead -- and with blocks shorter than a request's rows (8 at head_dim 64, 4 at 128), where every lane has an address of its own.
@pytest.mark.parametrize("D,block,S,splits", [(64, 1, 960, 1), (64, 1, 3300, 1), (64, 4, 9000, 1), (64, 16, 33000, 2), (128, 2, 5000, 1)])
@pytest.mark.parametrize("n", [33, 150])
def test_table_slices_beyond_the_lds_ring_per_lane_addresses(D, block, S, splits, n, monkeypatch):
    monkeypatch.setattr(W, "BLOCK_TOKENS", block)
    par = W.random_tree(np.random.default_rng(S), n, 4, 7, False)[0]
    case = W.custom_case(4250 + S, "bf16", 1, 2, 2, D, 500, [S], [par], paged=True, q_scale=2.0)
    case.block_size = block
    run_case(case, rows=sample_rows(case, 60), options={"splits": splits, "attn_impl": 2}, what=f"D={D} block {block} S={S}")


# blocks that are no power of two: the scalar kernel, with the split count cut to what its partial states have room for
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("S,splits", [(40, 0), (3000, 40), (6000, 0)])
def test_blocks_that_are_no_power_of_two(D, S, splits, monkeypatch):
    monkeypatch.setattr(W, "BLOCK_TOKENS", 24)
    par = W.random_tree(np.random.default_rng(S), 16, 4, 7, False)[0]
    case = W.custom_case(4300 + S, "bf16", 1, 4, 1, D, 500, [S], [par], paged=True, q_scale=2.0)
    case.block_size = 24
    run_case(case, rows=sample_rows(case, 60), options={"splits": splits}, what=f"block 24 D={D} S={S}")


@pytest.mark.parametrize("dtype,hq,hkv,d,n", [("bf16", 4, 4, 128, 20), ("bf16", 8, 2, 128, 100), ("bf16", 4, 4, 64, 30), ("f32", 4, 2, 64, 9)])
@pytest.mark.parametrize("blocks", [2 ** 31 - 1, 2 ** 31, 2 ** 33 + 3])
def test_pools_that_are_said_to_be_larger_than_an_entry_can_name(dtype, hq, hkv, d, n, blocks):
    """The size only bounds entries, so with a valid table the results are those of the true one."""
    import torch
    print(f"[case] pool of {blocks} blocks {dtype} {hq}/{hkv} x {d}", flush=True)
    case = W.custom_case(4400 + n, dtype, 2, hq, hkv, d, 300, [300, 40], [W.random_tree(np.random.default_rng(n + b), n, 3, 7, False)[0] for b in range(2)],
                         paged=True, p_match=0.9)
    got = []
    for size in (None, blocks):
        dc, ver = B.DeviceCase(case), B.Verifier(B.config_for_case(case))
        if size:
            dc.kv.capacity_or_num_blocks = size
        out, acc_len, acc_tok = ver.verify_tree(dc.q, dc.kv, case.kv_len, case.node_offsets, case.parent, case.tokens, dc.logits)
        ver.compact_kv([dc.kv], 2)
        torch.cuda.synchronize()
        got.append((out.clone(), dc.k, dc.v, torch.from_numpy(acc_len), torch.from_numpy(acc_tok)))
        ver.close()
    assert all(torch.equal(a, b) for a, b in zip(*got))
