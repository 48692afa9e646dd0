"""The logits scan and the acceptance at the sizes where they can go wrong: rows that start anywhere inside a
16-byte piece, chunks of a few elements, maxima in the pieces' rests and in several chunks, more nodes than a
wavefront has lanes, chains as long as the tree; in the attention's launch and as a launch of its own."""
import numpy as np
import pytest

from paper_2511_21699_amd import workloads as W
from tests.gpu_harness import run_case, sample_rows

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fuse", [1, 0])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("V", [1, 5, 8, 9, 1023, 8192, 8193, 8199, 16391, 33333])
def test_first_maximum_of_rows_at_any_alignment(V, dtype, fuse):
    rng = np.random.default_rng(V)
    par = W.random_tree(rng, 37, 4, 6, False)[0]
    case = W.custom_case(300 + V, dtype, 1, 2, 2, 128, V, [20], [par], p_match=0.8)
    x = np.round(rng.standard_normal(case.logits.shape, dtype=np.float32) * 2) / 2      # many equal maxima
    for i in range(37):                                                                 # a unique one anywhere, edges first
        if i % 3:
            x[i, [0, V - 1, min(V - 1, 8191), min(V - 1, 8192), int(rng.integers(V))][i % 5]] = 9.0
    x[3] = -3.0e38
    x[4, :] = -0.0
    x[4, V // 2] = 0.0
    case.logits = W.f32_to_bf16_bits(x) if dtype == "bf16" else x
    run_case(case, options={"fuse_logits": fuse}, what=f"V={V} {dtype}")


@pytest.mark.parametrize("N", [64, 65, 128, 129, 255, 256])
@pytest.mark.parametrize("shape", ["chain", "star", "random"])
def test_acceptance_of_trees_beyond_a_wavefront(N, shape):
    rng = np.random.default_rng(N)
    pars = [W.chain_tree(N) if shape == "chain" else W.star_tree(N) if shape == "star" else W.random_tree(rng, N, 3, 9, False)[0],
            W.chain_tree(3)]
    for p in (0.6, 0.99, 1.0):
        case = W.custom_case(400 + N, "bf16", 2, 2, 2, 128, 700, [33, 5], pars, p_match=p)
        run_case(case, rows=sample_rows(case, 16), what=f"{shape} {N} p={p}")


# the stand-alone scan with short chunks (at most 1024 whole ones) around a short chunk's edges, and on either side of that line
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("N,V", [(3, 2047), (3, 2048), (3, 2049), (5, 6151), (128, 65536), (129, 65535), (129, 65537)])
def test_scan_with_short_chunks(N, V, dtype):
    rng = np.random.default_rng(N + V)
    par = W.random_tree(rng, N, 4, 7, False)[0]
    case = W.custom_case(500 + N + V, dtype, 1, 2, 2, 128, V, [20], [par], p_match=0.8)
    x = np.zeros(case.logits.shape, dtype=np.float32)
    for i in range(N):  # pairs of equal maxima on either side of an edge, or far apart
        a = [0, 2047, 2048, V - 1, int(rng.integers(V))][i % 5]
        x[i, [min(a, V - 1), min(a + 1, V - 1), int(rng.integers(V))]] = 5.0
    case.logits = W.f32_to_bf16_bits(x) if dtype == "bf16" else x
    run_case(case, rows=sample_rows(case, 8), options={"fuse_logits": 0}, what=f"N={N} V={V} {dtype}")


# workgroups of the one-launch verification that do the logits work: the fewest, more than there are items for, the most; in one
# round of attention workgroups and in several, and beside the fp32 kernel
@pytest.mark.parametrize("wgs", [8, 40, 192])
@pytest.mark.parametrize("dtype,heads,lens", [("bf16", 4, [700, 90]), ("bf16", 32, [300] * 12), ("f32", 4, [200, 33])])
def test_any_number_of_logits_workgroups(wgs, dtype, heads, lens):
    rng = np.random.default_rng(wgs)
    pars = [W.random_tree(rng, 20 + 3 * i, 4, 6, False)[0] for i in range(len(lens))]
    case = W.custom_case(600 + wgs + heads, dtype, len(lens), heads, heads, 128, 9001, lens, pars, p_match=0.8)
    run_case(case, rows=sample_rows(case, 60), options={"logits_wgs": wgs}, what=f"{wgs} workgroups {dtype} {heads} heads")
