"""The fp32 attention on the matrix cores around its edges: tiles of 16 rows, units of 16 keys over 8 wavefronts, splits
merged by the last workgroup or by the merge kernel, verification in one launch and in several, paged caches of any
block size, and values that only some queries may see."""
import numpy as np
import pytest

from paper_2511_21699_amd import binding as B
from paper_2511_21699_amd import workloads as W
from tests.gpu_harness import run_case, sample_rows

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,g", [(1, 1), (15, 1), (16, 1), (17, 1), (8, 4), (64, 2), (256, 1)])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("S,options", [(0, {}), (1, {"splits": 1}), (15, {"fuse_logits": 0}), (127, {"splits": 2}),
                                       (700, {}), (1333, {"splits": 11}), (1333, {"splits": 3, "external_merge": 1})])
def test_tile_and_unit_edges(n, g, D, S, options):
    par = W.random_tree(np.random.default_rng(n + S), n, 4, 7, False)[0]
    case = W.custom_case(6100 + n + S, "f32", 1, 3 * g, 3, D, 300, [S], [par], q_scale=2.0)
    run_case(case, rows=sample_rows(case, 60), options=options, what=f"rows {n * g} D={D} S={S} {options}")


@pytest.mark.parametrize("impl", [0, 1])
@pytest.mark.parametrize("layout", [B.CB_LAYOUT_TOKEN_MAJOR, B.CB_LAYOUT_HEAD_MAJOR])
def test_ragged_paged_batch_beside_the_scalar_kernel(impl, layout):
    rng = np.random.default_rng(5)
    pars = [W.random_tree(rng, n, 4, 9, False)[0] for n in (40, 3, 65, 17)]
    case = W.custom_case(6200, "f32", 4, 16, 8, 128, 500, [900, 0, 33, 2100], pars, paged=True, q_scale=2.0)
    run_case(case, options={"attn_impl": impl}, layout=layout, what=f"ragged paged impl={impl}")


@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
def test_value_of_an_unseen_node_leaves_no_trace(bad):
    case = W.custom_case(6300, "f32", 1, 4, 2, 64, 100, [37], [W.star_tree(20)], p_match=0.0)
    case.v = case.v.copy()
    case.v[0, 37 + 9] = bad                                  # (only node 9 sees it)
    rows = np.asarray([(0, h, i) for h in range(4) for i in range(20) if i != 9], dtype=np.int32)
    run_case(case, rows=rows, compact=False, what=f"value {bad} at one leaf")
