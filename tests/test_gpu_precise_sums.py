"""bf16 calls that hold probabilities and partial sums in 32 bits (head_dim 64; head_dim 128 where a split's slice of
the block table has more than 1022 entries): the output's error against the float64 oracle is that of rounding the
result to bf16, and no larger than the scalar kernel's, which computes everything in fp32."""
import numpy as np
import pytest

from oracle import cb_oracle as O
from paper_2511_21699_amd import binding as B
from paper_2511_21699_amd import workloads as W
from tests.gpu_harness import structured_rows

pytestmark = pytest.mark.gpu

rng = np.random.default_rng(9)
tree = lambda n: W.random_tree(rng, n, 4, 8, False)[0]  # noqa: E731

CASES = [  # name, B, Hq, Hkv, D, lengths, trees, paged block (0: contiguous), splits
    ("one split", 1, 8, 8, 64, [300], [tree(30)], 0, 1),
    ("several splits", 1, 32, 8, 64, [3000], [tree(16)], 0, 8),
    ("tiles of 128 rows", 1, 8, 2, 64, [1500], [tree(32)], 0, 5),
    ("tiles of 256 rows and a rest", 1, 16, 2, 64, [900], [tree(40)], 0, 3),
    ("batch, paged", 3, 8, 4, 64, [700, 40, 333], [tree(20), tree(3), tree(45)], 16, 0),
    ("merge by the last workgroup", 24, 32, 32, 64, [500] * 24, [tree(9)] * 24, 0, 2),
    ("head_dim 128, table of 1100 entries, small tiles", 2, 8, 8, 128, [1090, 60], [tree(33), tree(5)], 1, 1),
    ("head_dim 128, two slices of 1100 entries, wide tiles", 1, 8, 2, 128, [2150], [tree(40)], 1, 2),
    # (the plan's slices are shorter, in 32 bits as the shape decides)
    ("head_dim 128, batch in slices of under 1022 entries, small tiles", 5, 32, 32, 128, [2500, 3000, 3500, 4000, 4500], [tree(9)] * 5, 1, 0),
    ("head_dim 128, batch in slices of under 1022 entries, wide tiles", 4, 64, 16, 128, [1600, 2100, 2600, 3100], [tree(70)] * 4, 1, 0),
]


@pytest.mark.parametrize("name,Bn,Hq,Hkv,D,lens,parents,bs,splits", CASES, ids=[c[0] for c in CASES])
def test_error_is_that_of_the_output_rounding(name, Bn, Hq, Hkv, D, lens, parents, bs, splits, monkeypatch):
    import torch
    monkeypatch.setattr(W, "BLOCK_TOKENS", bs)
    case = W.custom_case(4400 + D + max(lens), "bf16", Bn, Hq, Hkv, D, 64, lens, parents, paged=bs > 0, q_scale=2.0)
    case.block_size = bs
    rows = structured_rows(case)
    ref = O.attention_rows(case, rows, threads=16)
    floor = np.linalg.norm(W.to_f64(W.f32_to_bf16_bits(ref.astype(np.float32)), "bf16") - ref)
    err = {}
    for impl in (0, 1):
        dc = B.DeviceCase(case)
        ver = B.Verifier(B.config_for_case(case))
        ver.set_option("attn_impl", impl)
        ver.set_option("splits", splits)
        print(f"[precise] {name}: implementation {impl}", flush=True)
        try:
            out, _, _ = ver.verify_tree(dc.q, dc.kv, case.kv_len, case.node_offsets, case.parent, case.tokens, dc.logits)
            torch.cuda.synchronize()
            if impl == 0:
                assert ver.last_launch_info()["impl"] == 2
        finally:
            ver.close()
        got = W.to_f64(B.to_host(out, "bf16"), "bf16")
        err[impl] = np.linalg.norm(np.stack([got[case.node_offsets[b] + i, h] for b, h, i in rows]) - ref)
    # Beside the output's rounding (2^-9) there are the two-term probabilities (2^-17) and fp32 sums: they move the norm by
    # far less than a hundredth.  (bf16 probabilities and partial sums would add two roundings of the output's size.)
    assert err[0] <= 1.01 * floor, (err, floor)
    assert err[0] <= 1.01 * err[1], (err, floor)
