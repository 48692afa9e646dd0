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


# (splits, 32-key units that make them real: rounded up to whole units a split's keys give that number of splits) x how they are
# merged: cooperatively, by the last to arrive, by a kernel, cooperatively but every workgroup gives up.  A bf16 merge has up to 16
# slots in flight: 9 and 14 leave part of a batch, 17 and 31 take a second one.  The 128 pieces of 244 rows at head_dim 128 are merged
# four at a time up to 15 splits, two beyond.
@pytest.mark.parametrize("splits,units", [(2, 62), (4, 62), (9, 63), (14, 56), (17, 51), (31, 62)])
@pytest.mark.parametrize("options,merge", [({}, "cooperative"), ({"coop_merge": 0}, None), ({"external_merge": 1}, "merge_kernel"),
                                           ({"merge_spin_limit": 0}, "cooperative")])
@pytest.mark.parametrize("D,n,g", [(128, 61, 4), (128, 90, 1), (64, 75, 3)])
def test_merges_of_wide_tiles(splits, units, options, merge, D, n, g):
    par = W.random_tree(np.random.default_rng(splits), n, 4, 7, False)[0]
    case = W.custom_case(5900 + splits, "bf16", 1, 2 * g, 2, D, 300, [32 * units - n], [par], q_scale=2.0)
    info = run_case(case, rows=sample_rows(case, 60), options=dict(options, splits=splits), what=f"{splits} splits {options} D={D} rows {n * g}")["info"]
    if merge is None:  # (a tile's partial states beyond 320 KiB go to the kernel: what one workgroup would pull takes longer)
        tile = 32 * D * (4 if D == 64 else 2) + 32 * 8
        merge = "merge_kernel" if splits * -(-n * g // 32) * tile > 320 * 1024 else "last_arrival"
    assert (info["nsplit"], info["merge"]) == (splits, merge), info


# tiles of 65 to 128 rows: sweeps on either side of the lengths beyond which a wave takes two row tiles (2048 keys of a paged cache
# with more than 96 rows, 4096 in a batch), and tiles of one row more than a wave's share
@pytest.mark.parametrize("rows", [65, 96, 97, 128])
@pytest.mark.parametrize("batch,keys,paged", [(1, 2048, True), (1, 2049, True), (1, 2100, False), (2, 4096, False), (2, 4097, False), (2, 4128, True)])
def test_sweeps_of_up_to_128_rows(rows, batch, keys, paged):
    pars = [W.random_tree(np.random.default_rng(rows + b), rows if b == 0 else 71, 4, 7, False)[0] for b in range(batch)]
    lens = [keys - rows] + [1300] * (batch - 1)
    case = W.custom_case(6100 + rows, "bf16", batch, 2, 2, 128, 300, lens, pars, paged=paged, q_scale=2.0)
    run_case(case, rows=sample_rows(case, 80), options={"splits": 1}, what=f"{rows} rows, {batch} sequences, {keys} keys, paged {paged}")
