"""Row tiles of the MFMA attention around their edges: up to 64 rows in one small tile, up to 128 and up to 256 in the
two forms of the wide one, more in several; head_dim 64 and 128."""
import numpy as np
import pytest

from paper_2511_21699_amd import binding as B
from paper_2511_21699_amd import workloads as W
from tests.gpu_harness import run_case, sample_rows

pytestmark = pytest.mark.gpu


# nodes x query heads per kv head = rows of a tile; prefixes of a few keys, around a unit of 32, and enough for the
# unmasked part of the sweep
@pytest.mark.parametrize("n,g", [(1, 1), (17, 1), (64, 1), (65, 1), (32, 4), (129, 1), (64, 4), (86, 3), (150, 4)])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("S,splits", [(3, 1), (31, 1), (700, 1), (1333, 3)])
def test_row_tile_edges(n, g, D, S, splits):
    par = W.random_tree(np.random.default_rng(n + S), n, 4, 7, False)[0]
    case = W.custom_case(5200 + n + S, "bf16", 1, 2 * g, 2, D, 500, [S], [par], paged=False, q_scale=2.0)
    run_case(case, rows=sample_rows(case, 50), options={"splits": splits, "attn_impl": 2}, what=f"rows {n * g} D={D} S={S}")


# One launch whose sequences have tiles of every kind (up to 32, 64, 96, 128, 256 rows, several tiles), paged and in both layouts
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("paged,layout", [(True, B.CB_LAYOUT_TOKEN_MAJOR), (True, B.CB_LAYOUT_HEAD_MAJOR), (False, B.CB_LAYOUT_HEAD_MAJOR)])
@pytest.mark.parametrize("splits", [0, 1, 3])
def test_sequences_with_tiles_of_every_kind(D, paged, layout, splits):
    rng = np.random.default_rng(D + splits)
    sizes, lens = [9, 16, 17, 32, 33, 48, 64, 100, 150], [700, 31, 433, 1000, 90, 1500, 257, 640, 801]
    pars = [W.random_tree(rng, n, 4, 7, False)[0] for n in sizes]
    case = W.custom_case(5300 + D, "bf16", len(sizes), 4, 2, D, 500, lens, pars, paged=paged, q_scale=2.0)
    run_case(case, rows=sample_rows(case, 120), layout=layout, options={"splits": splits, "attn_impl": 2}, what=f"D={D} paged={paged} splits={splits}")
