"""Launch planning, on the host alone: what a call's shape decides whatever split count the planner finds fastest."""
import ctypes as C

import numpy as np
import pytest

from paper_2511_21699_amd import binding as B


def plan(hq, hkv, lens, nodes, block=0, vocab=32000, verification=True, d=128, logits="bf16"):
    """nodes: one size for all sequences, or one each."""
    n = np.broadcast_to(np.asarray(nodes, dtype=np.int32), len(lens))
    cfg = B.make_config(hq, hkv, d, "bf16", logits, len(lens), int(n.max()), 8, vocab, block)
    a = np.asarray(lens, dtype=np.int32)
    offs = np.concatenate([[0], np.cumsum(n)]).astype(np.int32)
    out = (C.c_int32 * 6)()
    ip = lambda x: x.ctypes.data_as(C.POINTER(C.c_int32))  # noqa: E731
    assert B.load().cb_debug_plan(C.byref(cfg), len(lens), ip(a), ip(offs), int(verification), out) == 0
    return dict(zip(("impl", "nsplit", "chunk", "precise", "logits_wgs", "fused"), out))


def steps(lo, step, batch):
    return [lo + step * b for b in range(batch)]


# Plans of fewer and longer splits put these calls' sums in 32 bits: slices of the block table beyond 1022 entries.
LONG_SLICES = [  # heads, kv heads, block, lengths, nodes, verification
    (32, 32, 8, steps(8100, 5700, 10), 64, False), (40, 40, 16, steps(9600, 5000, 11), 16, False), (8, 8, 16, steps(22800, 3000, 11), 4, False),
    (8, 8, 8, steps(11700, 4000, 13), 128, False), (32, 32, 8, steps(27900, 200, 8), 230, True), (32, 8, 16, steps(27300, 5000, 9), 128, True),
    (40, 40, 16, steps(10500, 3400, 13), 4, True), (8, 8, 8, steps(11100, 2100, 11), 230, True), (64, 8, 8, [36247], 230, True)]


@pytest.mark.parametrize("hq,hkv,block,lens,nodes,verification", LONG_SLICES)
def test_sums_stay_in_32_bits_whatever_the_splits(hq, hkv, block, lens, nodes, verification):
    p = plan(hq, hkv, lens, nodes, block, verification=verification)
    assert p["impl"] == 2 and p["precise"] == 1, p


def test_sums_of_short_slices_are_in_16_bits():
    assert plan(32, 32, [4111], 63, 16)["precise"] == 0
    assert plan(32, 8, steps(3000, 800, 12), 64, 16)["precise"] == 0


# Batches whose sums stay in the accumulators to the end: one split each.  (Partial states would round them to bf16.)
WHOLE = [  # heads, kv heads, lengths, nodes, verification
    (32, 32, steps(2700, 200, 12), 4, False), (40, 40, steps(3300, 800, 8), 4, False), (40, 40, steps(4200, 600, 6), 230, True),
    (40, 40, steps(7200, 400, 6), 128, True), (64, 8, steps(3600, 600, 4), 230, True), (64, 8, steps(7800, 200, 8), 128, True),
    (64, 8, steps(3000, 500, 8), 128, True)]


@pytest.mark.parametrize("block", [0, 16])
@pytest.mark.parametrize("hq,hkv,lens,nodes,verification", WHOLE)
def test_sequences_that_fill_the_chip_are_not_split(hq, hkv, lens, nodes, verification, block):
    assert plan(hq, hkv, lens, nodes, block, verification=verification)["nsplit"] == 1


# One sequence with wide tiles: a launch of one round, the logits' workgroups among them, merges its splits cooperatively.  (In
# two rounds, or with the chip half empty, these were slower than with a launch for the logits in front.)
@pytest.mark.parametrize("hq,hkv,length,nodes,vocab,logits", [
    (40, 40, 3303, 72, 128256, "bf16"), (40, 40, 4539, 116, 33333, "bf16"), (32, 8, 3183, 220, 32000, "f32"), (32, 32, 1759, 170, 32000, "bf16"),
    (40, 40, 987, 120, 32000, "f32"), (32, 8, 8192, 128, 32000, "bf16"), (40, 40, 65536, 256, 128256, "bf16")])
def test_one_sequence_stays_in_one_round(hq, hkv, length, nodes, vocab, logits):
    p = plan(hq, hkv, [length], nodes, vocab=vocab, logits=logits)
    grid = -(-nodes * (hq // hkv) // 256) * hkv * p["nsplit"] + p["logits_wgs"]
    assert p["fused"] and 200 <= grid <= 256, p


def test_batches_do_not_split_less_for_the_logits():
    # as many workgroups as compute units: the logits go in front, instead of a second round
    p = plan(32, 32, steps(1829 - 7 * 60, 60, 8), steps(155, 10, 8))
    assert (p["nsplit"], p["fused"]) == (1, 0), p
    # three splits each, in a round that leaves no units for the logits
    assert plan(32, 8, [5247, 1919, 4943, 2931, 2578, 2294], [92, 92, 92, 92, 92, 92], vocab=33333)["nsplit"] == 3


def test_short_logits_rows_get_workgroups_by_their_number():
    """A wave's round trip for each row bounds short rows, whatever few bytes they have."""
    lens, nodes = steps(40, 84, 16), steps(60, 9, 16)
    short, long_rows = plan(32, 32, lens, nodes, vocab=1000), plan(32, 32, lens, nodes, vocab=8000)
    assert short["fused"] and 16 <= short["logits_wgs"] <= 96, short
    assert long_rows["logits_wgs"] >= short["logits_wgs"]


def layers_plan(layers, hq, hkv, lens, nodes, block=0, vocab=32000, d=128):
    n = np.broadcast_to(np.asarray(nodes, dtype=np.int32), len(lens)).astype(np.int32)
    cfg = B.make_config(hq, hkv, d, "bf16", "bf16", len(lens), int(n.max()), 8, vocab, block)
    a, offs, out = np.asarray(lens, dtype=np.int32), np.concatenate([[0], np.cumsum(n)]).astype(np.int32), (C.c_int32 * 6)()
    ip = lambda x: x.ctypes.data_as(C.POINTER(C.c_int32))  # noqa: E731
    assert B.load().cb_debug_layers(C.byref(cfg), layers, len(lens), ip(a), ip(offs), out) == 0
    return dict(zip(("together", "tile_rows", "nsplit", "chunk", "precise", "logits_wgs"), out))


def test_layers_go_together_where_that_is_faster():
    assert layers_plan(32, 32, 32, [2048], 64)["nsplit"] == 1                          # 1024 whole sequences fill the chip
    assert layers_plan(2, 8, 8, [3000], 33)["nsplit"] > 1                              # 16 do not
    assert not layers_plan(2, 32, 8, steps(4105 - 7 * 10, 10, 8), 180)["together"]     # few long tiles: one by one
