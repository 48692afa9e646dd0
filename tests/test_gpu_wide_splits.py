"""Wide tiles of the MFMA attention at the sizes where their sweep and merge can go wrong: splits of fewer units than the ring
holds, of just as many and a few more, with a rest in the last unit; caches whose blocks are shorter and longer than a
request; merges of two and four pieces to a wave."""
import numpy as np
import pytest

from paper_2511_21699_amd import workloads as W
from tests.gpu_harness import run_case, sample_rows

pytestmark = pytest.mark.gpu


# the ring holds 9 units of 32 keys at head_dim 128 and 16 at 64; 6 (10) are requested before the first wait
@pytest.mark.parametrize("n,g", [(80, 1), (33, 4), (50, 5)])
@pytest.mark.parametrize("D,units", [(128, u) for u in (3, 5, 6, 7, 8, 9, 10, 11, 18)] + [(64, u) for u in (9, 10, 11, 13, 14, 15, 16, 17, 30)])
def test_splits_around_the_ring(D, units, n, g):
    par = W.random_tree(np.random.default_rng(n + units), n, 4, 7, False)[0]
    S = max(0, 32 * units - n - (0, 1, 31)[units % 3])
    case = W.custom_case(5700 + units, "bf16", 1, 2 * g, 2, D, 300, [S], [par], q_scale=2.0)
    run_case(case, rows=sample_rows(case, 50), options={"splits": 1}, what=f"rows {n * g} D={D} {units} units")


@pytest.mark.parametrize("block", [1, 4, 8, 32, 256])
@pytest.mark.parametrize("D,n,g", [(128, 70, 1), (128, 40, 4), (64, 70, 2)])
def test_blocks_beside_a_request(block, D, n, g, monkeypatch):
    monkeypatch.setattr(W, "BLOCK_TOKENS", block)
    par = W.random_tree(np.random.default_rng(block), n, 4, 7, False)[0]
    case = W.custom_case(5800 + block, "bf16", 2, 2 * g, 2, D, 300, [1111, 77], [par, W.chain_tree(5)], paged=True, q_scale=2.0)
    case.block_size = block
    run_case(case, rows=sample_rows(case, 60), options={"splits": 2}, what=f"block {block} D={D} rows {n * g}")


# splits of the tile x how they are merged: cooperatively (two pieces each, four, several rounds), by the last to arrive, by a kernel
@pytest.mark.parametrize("splits", [2, 4, 9, 17, 30])
@pytest.mark.parametrize("options", [{}, {"coop_merge": 0}, {"external_merge": 1}, {"merge_spin_limit": 0}])
@pytest.mark.parametrize("D,n,g", [(128, 61, 4), (128, 90, 1), (64, 75, 3)])
def test_merges_of_wide_tiles(splits, options, D, n, g):
    par = W.random_tree(np.random.default_rng(splits), n, 4, 7, False)[0]
    case = W.custom_case(5900 + splits, "bf16", 1, 2 * g, 2, D, 300, [32 * 31 - n], [par], q_scale=2.0)
    run_case(case, rows=sample_rows(case, 60), options=dict(options, splits=splits), what=f"{splits} splits {options} D={D} rows {n * g}")
