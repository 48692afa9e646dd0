"""Host-side check of the build's guard for loads issued as uninterpreted inline assembly
(build.untracked_load_violations): it accepts the kernel as compiled and catches a planted early use."""
import os
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


@pytest.mark.skipif(shutil.which("hipcc") is None, reason="needs hipcc")
def test_compiled_attention_kernel_passes():
    asm = build.device_asm(os.path.join(build.CSRC, "cb_attn_mfma.hip"))
    assert asm.count("global_load_lds_dwordx4") > 50          # the ring's requests are there, as inline assembly
    assert build.untracked_load_violations(asm) == []
    res = build.kernel_resources(asm)
    attn = {k: v for k, v in res.items() if "k_attn_mfma" in k or "k_verify_mfma" in k}
    assert len(attn) == 8                                      # four variants, each with and without the timeline stamps
    assert build.scratch_violations(asm) == []
    assert all(v[0] <= 256 for v in attn.values())             # two waves per SIMD


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
@pytest.mark.parametrize("name", ["cb_attn_mfma.hip", "cb_attn_wide.hip"])
def test_compiled_requests_keep_their_distance_from_the_base(name):
    asm = build.device_asm(os.path.join(build.CSRC, name))
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
