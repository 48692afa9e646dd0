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
