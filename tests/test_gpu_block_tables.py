"""Paged caches whose table slice of one split is longer than the part of it that the attention kernel keeps in
LDS at a time (1024 entries): the ring of table segments is refilled during the sweep."""
import numpy as np
import pytest

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
