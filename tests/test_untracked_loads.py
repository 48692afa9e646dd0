"""Host-side check of the build's guard for loads issued as uninterpreted inline assembly
(build.untracked_load_violations): it accepts the kernel as compiled and catches a planted early use."""
import functools
import os
import re
import shutil

import pytest

from paper_2511_21699_amd import build

LISTING = """
\ts_mov_b32 s0, 0
\t;;#ASMSTART
\tglobal_load_dwordx4 v[6:9], v[2:3], off
\t;;#ASMEND
\tv_or_b32_e32 v2, 0x200, v0
%s
\ts_waitcnt vmcnt(8)
\ts_barrier
\tv_mfma_f32_16x16x32_bf16 v[56:59], v[56:59], v[6:9], 0
"""


def test_checker_accepts_a_wait_before_the_first_use():
    assert build.untracked_load_violations(LISTING % "\tv_add_u32_e32 v10, v11, v12") == []


@pytest.mark.parametrize("early", ["\tv_mov_b32_e32 v40, v7", "\tv_mov_b64_e32 v[40:41], v[8:9]",
                                   "\tbuffer_store_dword v6, off, s[0:3], 0 offset:4",
                                   "\tv_accvgpr_write_b32 a0, v9"])
def test_checker_reports_a_use_before_the_wait(early):
    bad = build.untracked_load_violations(LISTING % early)
    assert len(bad) == 1 and "global_load_dwordx4 v[6:9]" in bad[0][1]


def test_checker_ignores_loads_the_compiler_tracks():
    text = "\tglobal_load_dwordx4 v[6:9], v[2:3], off\n\tv_mov_b32_e32 v40, v7\n"
    assert build.untracked_load_violations(text) == []


BRANCHES = """
\t;;#ASMSTART
\tglobal_load_dwordx4 v[6:9], v[2:3], off
\t;;#ASMEND
\ts_mov_b64 s[2:3], -1
\ts_cbranch_scc1 .LBB0_2
\ts_waitcnt vmcnt(4)
\ts_mov_b64 s[2:3], 0
.LBB0_2:
%s\ts_andn2_b64 vcc, exec, s[2:3]
\ts_cbranch_vccnz .LBB0_4
\ts_waitcnt vmcnt(0)
.LBB0_4:
\tv_accvgpr_write_b32 a0, v7
\ts_endpgm
"""


def test_checker_follows_both_sides_of_a_branch():
    wait, skipped = "\ts_waitcnt vmcnt(0)\n", "\ts_cbranch_execz .LBB0_9\n\ts_waitcnt vmcnt(0)\n.LBB0_9:\n"
    body = "\t;;#ASMSTART\n\tglobal_load_dwordx4 v[6:9], v[2:3], off\n\t;;#ASMEND\n%s\tv_mov_b32_e32 v40, v7\n\ts_endpgm\n"
    assert build.untracked_load_violations(body % wait) == []
    assert len(build.untracked_load_violations(body % skipped)) == 1
    assert len(build.untracked_load_violations(body % "\ts_branch .LBB0_9\n\ts_waitcnt vmcnt(0)\n.LBB0_9:\n")) == 1
    loop = ".LBB0_9:\n\tv_add_u32_e32 v10, v11, v12\n\ts_cbranch_scc1 .LBB0_9\n"
    assert build.untracked_load_violations(body % (loop + wait)) == []
    assert len(build.untracked_load_violations(body % loop)) == 1
    far = "\ts_getpc_b64 s[8:9]\n.Lpost_getpc0:\n\ts_add_u32 s8, s8, (.LBB0_9-.Lpost_getpc0)&4294967295\n\ts_setpc_b64 s[8:9]\n" + wait + ".LBB0_9:\n"
    assert len(build.untracked_load_violations(body % far)) == 1


@pytest.mark.parametrize("between,ok", [("", True), ("\ts_mov_b64 s[2:3], 0\n", False), ("\ts_xor_b64 s[2:3], s[2:3], s[4:5]\n", False),
                                        ("\tv_cmp_lt_i32_e64 s[2:3], -1, v51\n", False), ("\ts_mov_b32 s3, s8\n", False), ("\ts_mov_b64 s[4:5], 0\n", True)])
def test_checker_knows_a_flag_that_skips_a_wait_already_made(between, ok):
    assert (build.untracked_load_violations(BRANCHES % between) == []) == ok


@functools.lru_cache(maxsize=None)
def _asm(name):
    return build.device_asm(os.path.join(build.CSRC, name))


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_compiled_attention_kernel_passes():
    asm = _asm("cb_attn_mfma.hip")
    assert asm.count("global_load_lds_dwordx4") > 50          # the ring's requests are there, as inline assembly
    assert build.untracked_load_violations(asm) == []
    res = build.kernel_resources(asm)
    attn = {k: v for k, v in res.items() if "k_attn_mfma" in k or "k_verify_mfma" in k}
    assert len(attn) == 8                                      # four variants, each with and without the timeline stamps
    assert build.scratch_violations(asm) == []
    assert all(v[0] <= 256 for v in attn.values())             # two waves per SIMD


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
@pytest.mark.parametrize("name,kernels", [("cb_attn_wide.hip", 16), ("cb_attn_wide_px.hip", 16)])
def test_compiled_wide_kernel_passes(name, kernels):
    """Its queries go to accumulation registers: behind the ring's wait, never in front of it."""
    asm = _asm(name)
    assert asm.count("global_load_lds_dwordx4") > 50
    assert build.untracked_load_violations(asm) == [] and build.scalar_base_violations(asm) == []
    res = build.kernel_resources(asm)
    assert len(res) == kernels                                 # tiles to a wave or head_dim, contiguous or paged, alone or with the logits, timeline
    assert build.scratch_violations(asm, name) == []
    assert all(v[0] <= 512 for v in res.values())              # one wave per SIMD
    # the first kernel's first query register moved to an accumulation register in front of its wait, in the common block
    # behind a loop or at the load
    lines = asm.split("\n")
    load = next(i for i, c in enumerate(lines) if re.search(r"global_load_dwordx4 v\[\d+:\d+\]", c) and "ASMSTART" in lines[i - 1])
    reg = re.search(r"v\[(\d+):", lines[load])[1]
    last = next(i for i in range(load, len(lines)) if re.search(rf"v_accvgpr_write_b32 a\d+, v{reg}\b", lines[i]))
    wait = max(i for i in range(load, last) if re.match(r"\s*s_waitcnt vmcnt", lines[i]))
    for at in (load + 2, max(i for i in range(load, wait) if re.match(r"\.LBB", lines[i])) + 1):
        planted = lines[:at] + [f"\tv_accvgpr_write_b32 a200, v{reg}"] + lines[at:]
        bad = build.untracked_load_violations("\n".join(planted))
        assert load + 1 in [line for line, _ in bad], at


def test_scratch_checker_reports_spills():
    meta = """
  - .name:           k_good
    .private_segment_fixed_size: 0
    .vgpr_count:     200
    .vgpr_spill_count: 0
  - .name:           k_spills
    .private_segment_fixed_size: 864
    .vgpr_count:     256
    .vgpr_spill_count: 216
"""
    assert build.kernel_resources(meta) == {"k_good": (200, 0, 0), "k_spills": (256, 216, 864)}
    assert [k for k, _ in build.scratch_violations(meta)] == ["k_spills"]
    kept = meta.replace("864", "0")                            # registers kept in others
    assert [k for k, _ in build.scratch_violations(kept, "cb_attn_mfma.hip")] == ["k_spills"]
    assert build.scratch_violations(kept, "cb_attn_wide.hip") == []


BASE_LISTING = """
\tv_readfirstlane_b32 s6, v18
\t;;#ASMSTART
\ts_mov_b32 m0, s41
\ts_mov_b32 exec_lo, s12
\ts_mov_b32 exec_hi, s12
%s\tglobal_load_lds_dwordx4 v184, s[6:7]
\ts_mov_b64 exec, -1
\t;;#ASMEND
"""


@pytest.mark.parametrize("between,ok", [("", False), ("\ts_nop 0\n", False), ("\ts_nop 1\n", True), ("\ts_nop 0\n\ts_nop 0\n", True)])
def test_checker_counts_wait_states_before_a_scalar_base(between, ok):
    bad = build.scalar_base_violations(BASE_LISTING % between)
    assert (bad == []) == ok
    if not ok:
        assert "s[6:7]" in bad[0][1]


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
@pytest.mark.parametrize("name", ["cb_attn_mfma.hip"])  # (the wide kernel's requests have no scalar base)
def test_compiled_requests_keep_their_distance_from_the_base(name):
    asm = _asm(name)
    assert asm.count(", s[") > 0 and "global_load_lds_dwordx4" in asm
    assert build.scalar_base_violations(asm) == []


# The logits scan launches up to 1024 workgroups of 4 waves and counts on all of them being resident: four to a compute unit, a
# wave of each on every SIMD.  In the fp32 verification the scan must not take the attention's occupancy at head_dim 64.
@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
@pytest.mark.parametrize("name,kernel", [("cb_small_kernels.hip", "k_logits"), ("cb_attn_f32.hip", "k_verify_f32ILi64")])
def test_registers_leave_room_for_four_waves_per_simd(name, kernel):
    res = build.kernel_resources(build.device_asm(os.path.join(build.CSRC, name)))
    counts = [v[0] for k, v in res.items() if kernel in k]
    assert counts and max(counts) <= 128, res


# The fp32 kernels count on two workgroups of 8 waves to a compute unit at head_dim 64, and on half of the next one's waves at 128.
@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_registers_of_the_fp32_kernels():
    res = build.kernel_resources(_asm("cb_attn_f32.hip"))
    for d, most in ((64, 128), (128, 168)):
        counts = {k: v[0] for k, v in res.items() if f"f32ILi{d}" in k}
        assert len(counts) == 4 and max(counts.values()) <= most, counts
