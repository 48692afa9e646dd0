"""Calls whose rows go into shorter tiles than a kv head has rows: the option against the oracle, and what the planner may choose."""
import ctypes as C

import numpy as np
import pytest

from paper_2511_21699_amd import binding as B
from paper_2511_21699_amd import workloads as W
from .gpu_harness import run_case, structured_rows

CASES = [  # heads, kv heads, head_dim, prefixes, tree sizes, tile rows, other options, paged
    (8, 8, 128, [200], [65], 64, {}, False),                       # one row in the second tile
    (32, 8, 128, [500], [40], 64, {}, True),                       # 160 rows: 64, 64, 32
    (32, 8, 128, [500], [40], 128, {}, False),                     # 128, 32
    (16, 2, 128, [96, 700, 0], [33, 12, 1], 128, {}, False),       # 264, 96 and 8 rows
    (4, 4, 128, [1500], [256], 64, {}, False),
    (4, 4, 128, [1500], [256], 64, {"coop_merge": 0}, True),
    (4, 4, 128, [300], [256], 128, {"merge_spin_limit": 0}, True),
    (6, 3, 128, [100, 40], [100, 70], 64, {}, False),              # kv heads no multiple of 8
    (32, 8, 64, [700], [64], 64, {}, False),
    (32, 8, 64, [60, 800], [50, 17], 128, {}, True),
]


@pytest.mark.gpu
@pytest.mark.parametrize("i", range(len(CASES)))
def test_tiles_of_a_head(i):
    hq, hkv, d, lens, nodes, rows, options, paged = CASES[i]
    rng = np.random.default_rng(i)
    pars = [W.random_tree(rng, n, 3, 9, False)[0] for n in nodes]
    case = W.custom_case(8200 + i, "bf16", len(lens), hq, hkv, d, 700, lens, pars, paged=paged, p_match=0.8, q_scale=4.0 * d ** 0.5)
    run_case(case, rows=structured_rows(case), options=dict(options, tile_rows=rows), what=f"short tiles {i}")


def plans(hq, hkv, lens, nodes, block, verification, vocab=32000, d=128):
    n = np.broadcast_to(np.asarray(nodes, dtype=np.int32), len(lens))
    cfg = B.make_config(hq, hkv, d, "bf16", "bf16", len(lens), int(n.max()), 8, vocab, block)
    a = np.asarray(lens, dtype=np.int32)
    offs = np.concatenate([[0], np.cumsum(n)]).astype(np.int32)
    ip = lambda x: x.ctypes.data_as(C.POINTER(C.c_int32))  # noqa: E731
    got = []
    for f in (B.load().cb_debug_plan, B.load().cb_debug_tiles):
        out = (C.c_int32 * 6)()
        assert f(C.byref(cfg), len(lens), ip(a), ip(offs), int(verification), out) == 0
        got.append(list(out))
    return got


def test_shorter_tiles_keep_one_round_and_the_class_of_the_sums():
    rng = np.random.default_rng(5)
    shorter = 0
    for _ in range(600):
        hkv = int(rng.choice([2, 3, 8, 32, 40]))
        g, d = int(rng.choice([1, 2, 4, 8])), int(rng.choice([64, 128, 128]))
        lens = rng.integers(0, int(np.exp(rng.uniform(3, 10.5))), int(rng.choice([1, 1, 1, 2, 8])))
        nodes = rng.integers(1, int(rng.choice([20, 100, 256])) + 1, len(lens))
        block, ver = int(rng.choice([0, 2, 16])), bool(rng.integers(2))
        tall, p = plans(hkv * g, hkv, lens, nodes, block, ver, d=d)
        rows = int(nodes.max()) * g
        tallest = 64 if rows <= 64 else 256
        assert p[0] in (64, 128, 256) and p[0] <= tallest
        assert p[3] == tall[3] and (tall[1] > 1 or p[1] == 1)                  # what is in 32 bits, and what is not split
        if p[0] < tallest:
            shorter += 1
            assert p[5] + p[4] <= 256
            assert not (p[3] and d == 128)
        else:
            assert p[1] == tall[1] and p[2] == tall[2] and p[4] == tall[4]
    assert shorter > 100


# Slices of the block table that one split fewer would make longer than 16-bit sums go with.
LONG_TABLES = [  # heads, kv heads, lengths, nodes, block, verification
    (32, 32, [13169, 11104, 2591, 17612, 3498, 8277], [49, 33, 70, 82, 56, 45], 16, False), (40, 40, [23407] * 4, [119, 164, 179, 64], 16, True),
    (160, 40, [3980], [73], 2, False), (80, 40, [5580], [133], 2, True)]


@pytest.mark.parametrize("hq,hkv,lens,nodes,block,ver", LONG_TABLES)
def test_shorter_tiles_do_not_put_sums_in_32_bits(hq, hkv, lens, nodes, block, ver):
    tall, p = plans(hq, hkv, lens, nodes, block, ver)
    assert tall[3] == 0 and p[3] == 0, (tall, p)


@pytest.mark.parametrize("seed", range(8))
def test_sums_of_paged_calls_keep_their_class(seed):
    rng = np.random.default_rng(seed)
    for _ in range(250):
        hkv, g = int(rng.choice([8, 32, 40])), int(rng.choice([1, 2, 4, 8]))
        lens = rng.integers(1, int(np.exp(rng.uniform(6, 10.5))), int(rng.choice([1, 1, 2, 3, 6])))
        nodes = rng.integers(1, int(rng.choice([100, 256])) + 1, len(lens))
        block = int(rng.choice([1, 2, 4, 16]))
        alone, ver = [plans(hkv * g, hkv, lens, nodes, block, v) for v in (False, True)]
        for tall, p in (alone, ver):
            assert p[3] == tall[3]
        n = np.asarray(nodes, dtype=np.int32)
        cfg = B.make_config(hkv * g, hkv, 128, "bf16", "bf16", len(lens), int(n.max()), 8, 32000, block)
        a, offs, out = np.asarray(lens, dtype=np.int32), np.concatenate([[0], np.cumsum(n)]).astype(np.int32), (C.c_int32 * 6)()
        ip = lambda x: x.ctypes.data_as(C.POINTER(C.c_int32))  # noqa: E731
        assert B.load().cb_debug_layers(C.byref(cfg), int(rng.choice([2, 8, 32])), len(lens), ip(a), ip(offs), out) == 0
        assert not out[0] or out[4] == (alone[0][3] | ver[0][3])             # (a model's layers in one launch: as one by one)


# Two tiles to a head in three splits, whose merge has large slices, are no faster than one tile in more splits; one split, or more of them, are.
@pytest.mark.parametrize("hkv,length,nodes,tile", [(32, 790, 70, 256), (40, 790, 70, 256), (32, 800, 97, 256), (32, 800, 128, 256), (40, 800, 128, 256),
                                                   (40, 400, 70, 256), (32, 650, 96, 256), (32, 120, 66, 64), (8, 800, 97, 64), (16, 1000, 70, 64),
                                                   (32, 400, 97, 64), (8, 3200, 128, 64)])
def test_two_tiles_to_a_head(hkv, length, nodes, tile):
    assert plans(hkv, hkv, [length], [nodes], 0, True, vocab=1000)[1][0] == tile
