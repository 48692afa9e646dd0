"""Batches of sequences of unequal length and tile count: every workgroup that has keys is launched once, whatever number of
splits and row tiles its sequence has, with kv heads that are a multiple of 8 (only those workgroups are launched) and not."""
import numpy as np
import pytest

from paper_2511_21699_amd import workloads as W
from tests.gpu_harness import run_case, sample_rows

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hkv,g", [(8, 1), (16, 4), (8, 5), (4, 4), (2, 8), (3, 2)])
@pytest.mark.parametrize("sizes,lens", [([1, 64, 3, 64], [900, 0, 900, 31]), ([100, 7, 150], [5, 1300, 640]), ([256, 1], [64, 2000]),
                                        ([20] * 11, [37 * i for i in range(11)]),
                                        ([1 + 5 * i % 17 for i in range(64)], [29 * i * i % 641 for i in range(64)])])  # as many as a call can have
@pytest.mark.parametrize("splits", [0, 1, 5])
def test_every_tile_of_a_batch(hkv, g, sizes, lens, splits):
    rng = np.random.default_rng(len(sizes) + hkv)
    pars = [W.random_tree(rng, n, 4, 7, False)[0] for n in sizes]
    case = W.custom_case(6000 + hkv + g, "bf16", len(sizes), hkv * g, hkv, 128, 400, lens, pars, q_scale=2.0)
    run_case(case, rows=sample_rows(case, 150), options={"splits": splits}, what=f"{hkv} x {g} heads {sizes} splits={splits}")
