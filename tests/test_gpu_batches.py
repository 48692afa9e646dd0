"""Batches of sequences of unequal length and tile count: every workgroup that has keys is launched once, whatever number of
splits and row tiles its sequence has, with kv heads that are a multiple of 8 (only those workgroups are launched) and not."""
import numpy as np
import pytest

from paper_2511_21699_amd import workloads as W
from tests.gpu_harness import run_case, sample_rows
from tests.test_gpu_short_tiles import plans

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


# Jobs that fill the chip behind the logits' workgroups instead of beside them (planned so by the host: asserted), some in two splits.
BEHIND = [(32, 2, [106, 17, 391, 595, 712], [16, 15, 28, 19, 26], 300), (32, 1, [818, 301, 475, 527, 18], [23, 45, 37, 27, 23], 300),
          (40, 2, [97, 511, 34, 1006], [30, 23, 15, 11], 32000)]


@pytest.mark.parametrize("hkv,g,lens,sizes,vocab", BEHIND)
@pytest.mark.parametrize("paged", [False, True])
def test_batches_whose_jobs_are_behind_the_logits(hkv, g, lens, sizes, vocab, paged):
    tall, p = plans(hkv * g, hkv, lens, sizes, 16 if paged else 0, True, vocab=vocab)
    assert p[4] > 0 and 256 - p[4] < p[5] <= 256 and p[1] > 1, p
    rng = np.random.default_rng(len(sizes) + hkv)
    pars = [W.random_tree(rng, n, 4, 7, False)[0] for n in sizes]
    case = W.custom_case(6100 + hkv + g, "bf16", len(sizes), hkv * g, hkv, 128, vocab, lens, pars, paged=paged, q_scale=2.0, p_match=0.9)
    got = run_case(case, rows=sample_rows(case, 150), what=f"behind the logits {hkv} x {g} heads {sizes} paged={paged}")
    assert got["info"]["fused"] and got["info"]["nsplit"] == p[1] and got["info"]["chunk"] == p[2]
