"""Build libcacheback_verify.so for gfx950 with hipcc (in-tree, next to this file)."""
from __future__ import annotations

import glob
import os
import re
import subprocess
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libcacheback_verify.so")

FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-Wall", "-Wno-unused-function",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         # every atomic here is issued by one thread; the wave-aggregation pass would only add a
         # wait for the result right behind the atomic, where the kernels want it in flight
         "-mllvm", "-amdgpu-atomic-optimizer-strategy=None",
         "-I", os.path.join(ROOT, "include"), "-I", CSRC]

# The wide kernel's wavefronts have a SIMD to themselves and use more than 256 registers.  With matrix instructions in their
# form for accumulation registers the scores would be copied out of those before every vector instruction; in the other
# form only what the vector ALU rarely touches ends up there (the queries and what does not fit).
FILE_FLAGS = {name: ["-mllvm", "-amdgpu-mfma-vgpr-form=1"] for name in ("cb_attn_wide.hip", "cb_attn_wide_px.hip", "cb_attn_wide_layers.hip", "cb_attn_wide_step.hip")}


def _flags(src: str) -> list:
    return FLAGS + FILE_FLAGS.get(os.path.basename(src), [])


def _compile(src: str) -> str:
    obj = os.path.join(OBJ, os.path.basename(src) + ".o")
    subprocess.run(["hipcc", *_flags(src), "-c", src, "-o", obj], check=True)
    return obj


def device_asm(src: str) -> str:
    """The gfx950 assembly hipcc makes of one source file, with the library's flags."""
    os.makedirs(OBJ, exist_ok=True)
    out = os.path.join(OBJ, os.path.basename(src) + ".s")
    flags = [f for f in _flags(src) if f not in ("-fPIC",)]
    subprocess.run(["hipcc", *flags, "-S", "--offload-device-only", src, "-o", out], check=True,
                   stderr=subprocess.DEVNULL)
    with open(out) as f:
        return f.read()


_VREG = re.compile(r"\bv(?:\[(\d+):(\d+)\]|(\d+)\b)")
_SREG = re.compile(r"\bs(?:\[(\d+):(\d+)\]|(\d+)\b)")


def _ranges(pattern, code: str) -> list:
    return [(int(m[1]), int(m[2])) if m[1] else (int(m[3]), int(m[3])) for m in pattern.finditer(code)]


class _Listing:
    """The instructions of an assembly listing and where each can go on: `code` without comments, `jump(i)` the target of a
    branch (long ones are an s_setpc_b64 behind the address arithmetic that names the label), `falls(i)` whether the next line
    can follow."""

    def __init__(self, asm: str):
        self.code = [line.split(";")[0].strip() for line in asm.split("\n")]
        self.labels = {m[1]: i for i, c in enumerate(self.code) if (m := re.match(r"(\.?\w+):", c))}
        self.regs, self.sregs = {}, {}

    def jump(self, i: int):
        c = self.code[i]
        if m := re.match(r"s_c?branch\w* (\.?\w+)", c):
            return self.labels[m[1]]
        if c.startswith("s_setpc_b64"):
            for j in range(i - 1, max(i - 10, -1), -1):
                if m := re.search(r"(\.LBB\w+)-", self.code[j]):
                    return self.labels[m[1]]
            raise RuntimeError(f"line {i + 1}: jump to an unknown place")
        return None

    def falls(self, i: int) -> bool:
        return i + 1 < len(self.code) and not re.match(r"s_(branch|setpc_b64|endpgm)", self.code[i])

    def vregs(self, i: int) -> list:
        if i not in self.regs:
            self.regs[i] = _ranges(_VREG, self.code[i])
        return self.regs[i]

    def flags(self, i: int, known: frozenset) -> frozenset:
        """What line i makes of the scalar pairs known to hold 0 or -1 (and "vcc", known to be zero or not).  A wait that the
        source skips on a condition is often guarded by such a pair, set where the condition was evaluated."""
        c = self.code[i]
        if m := re.match(r"s_mov_b64 s\[(\d+):\d+\], (0|-1)$", c):
            lo = int(m[1])
            return frozenset([(k, v) for k, v in known if k == "vcc" or abs(k - lo) > 1] + [(lo, m[2] == "-1")])
        if not known or c.startswith("s_cbranch"):
            return known
        if m := re.match(r"s_(andn2|and)_b64 vcc, exec, s\[(\d+):\d+\]$", c):
            pairs = {k: v for k, v in known if k != "vcc"}
            if int(m[2]) in pairs:  # (some lane is active)
                pairs["vcc"] = pairs[int(m[2])] != (m[1] == "andn2")
            return frozenset(pairs.items())
        if i not in self.sregs:
            self.sregs[i] = _ranges(_SREG, c), "vcc" in c
        named, vcc = self.sregs[i]
        return frozenset((k, v) for k, v in known if (not vcc if k == "vcc" else not any(a <= k + 1 and b >= k for a, b in named)))


def untracked_load_violations(asm: str) -> list:
    """The attention kernels issue some loads as inline assembly the compiler does not know to be
    loads, and wait for them themselves before their first use.  That is only right while the compiler
    leaves the destination registers alone in between (a copy or a spill, to memory or to an accumulation register, would
    read them before the data is there).  For every such load (a global_load_dwordx4 inside an inline-assembly
    block) this follows the listing along both sides of every branch up to the first vmcnt wait, and reports
    the load if an instruction on the way names one of its registers.  Returns a list of (line number, text) pairs, empty if
    all is well."""
    lst = _Listing(asm)
    bad = []
    in_asm = False
    for i, line in enumerate(asm.split("\n")):
        if "ASMSTART" in line or "ASMEND" in line:
            in_asm = "ASMSTART" in line
            continue
        # (every register-returning load spelling: the query rows' and the logits item's 16-byte loads today)
        m = re.search(r"(?:global|buffer|flat)_load_dword(?:x[234])? v\[(\d+):(\d+)\]", line) if in_asm else None
        if not m:
            continue
        lo, hi = int(m.group(1)), int(m.group(2))
        seen, todo, touched = set(), [(i + 1, frozenset())] if lst.falls(i) else [], False
        while todo and not touched:
            j, known = todo.pop()
            if (j, known) in seen:
                continue
            seen.add((j, known))
            if lst.code[j].startswith("s_waitcnt") and "vmcnt" in lst.code[j]:
                continue
            touched = any(a <= hi and b >= lo for a, b in lst.vregs(j))
            after, target = lst.flags(j, known), lst.jump(j)
            vcc = dict(known).get("vcc") if re.match(r"s_cbranch_vccn?z", lst.code[j]) else None
            taken = None if vcc is None else vcc == lst.code[j].startswith("s_cbranch_vccnz")
            if target is not None and taken is not False:
                todo.append((target, after))
            if lst.falls(j) and taken is not True:
                todo.append((j + 1, after))
        if touched:
            bad.append((i + 1, line.strip()))
    return bad


def scalar_base_violations(asm: str) -> list:
    """Loads inside inline assembly whose address has a scalar base (global_load... vN, s[a:b]).  The chip
    wants five wait states between a vector instruction that writes a scalar register (v_readfirstlane_b32)
    and a load that reads it; the compiler keeps that rule for its own instructions but does not look inside
    inline assembly.  The statement may follow such a write directly, so it has to hold the five itself:
    every instruction in front of the load counts one, s_nop n counts n + 1.  Returns a list of (line number,
    text) pairs of the loads that come too early."""
    bad = []
    in_asm, states = False, 0
    for i, line in enumerate(asm.split("\n")):
        if "ASMSTART" in line or "ASMEND" in line:
            in_asm, states = "ASMSTART" in line, 0
            continue
        code = line.split(";")[0].strip()
        if not in_asm or not code:
            continue
        if re.match(r"(?:global|scratch|flat)_(?:load|store)\w* .*\bs\[\d+:\d+\]", code) and states < 5:
            bad.append((i + 1, code))
        nop = re.match(r"s_nop (\d+)", code)
        states += int(nop.group(1)) + 1 if nop else 1
    return bad


def kernel_resources(asm: str) -> dict:
    """{kernel symbol: (vgpr_count, vgpr_spill_count, private_segment_fixed_size)} from the listing's metadata."""
    out, name, cur = {}, None, {}
    for line in asm.split("\n"):
        m = re.match(r"\s*(?:- )?\.(name|vgpr_count|vgpr_spill_count|private_segment_fixed_size):\s*(\S+)", line)
        if not m:
            continue
        key, val = m.group(1), m.group(2)
        if key == "name":
            name = val
        else:
            cur[key] = int(val)
        if name and len(cur) == 3:
            out[name] = (cur["vgpr_count"], cur["vgpr_spill_count"], cur["private_segment_fixed_size"])
            name, cur = None, {}
    return out


def scratch_violations(asm: str, file_name: str = "") -> list:
    """Kernels of the listing that spill registers or use scratch memory.  In the attention kernel a spill
    reload from memory inside the K/V ring phase would be a compiler-generated load, and with it a wait for every load in
    flight, in a loop whose waits are counted by hand.  In files with flags of their own (FILE_FLAGS) the listing's spill count
    also holds vector registers kept in accumulation registers, which no memory access serves: there it is not looked at."""
    return [(k, v) for k, v in kernel_resources(asm).items() if v[2] != 0 or (v[1] != 0 and file_name not in FILE_FLAGS)]


def build(verbose: bool = False) -> str:
    os.makedirs(OBJ, exist_ok=True)
    srcs = sorted(glob.glob(os.path.join(CSRC, "*.hip")) + glob.glob(os.path.join(CSRC, "*.cpp")))
    checked = ["cb_attn_wide_px.hip", "cb_attn_wide.hip", "cb_attn_wide_layers.hip", "cb_attn_wide_step.hip", "cb_attn_mfma.hip"]
    with ThreadPoolExecutor(max_workers=min(8, len(srcs) + len(checked))) as ex:
        listings = [ex.submit(device_asm, os.path.join(CSRC, name)) for name in checked]  # (the longest first, beside the compilation)
        objs = list(ex.map(_compile, sorted(srcs, key=lambda s: os.path.basename(s) not in checked)))
    for name, listing in zip(checked, listings):
        asm = listing.result()
        bad = untracked_load_violations(asm)
        if bad:
            raise RuntimeError(f"{name}: registers of untracked loads are touched before their wait: {bad[:4]}")
        bad = scalar_base_violations(asm)
        if bad:
            raise RuntimeError(f"{name}: loads too close behind a possible write of their scalar base: {bad[:4]}")
        bad = scratch_violations(asm, name)
        if bad:
            raise RuntimeError(f"{name}: kernels that spill or use scratch memory: {bad[:4]}")
    subprocess.run(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB, *objs], check=True)
    if verbose:
        print(LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
