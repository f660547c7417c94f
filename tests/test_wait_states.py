"""CPU-side check of the built gfx950 code: wait states ahead of memory instructions.  The hardware does not wait by itself, and the compiler
does not see the loads that are written as inline assembly:
    an SGPR written by a vector instruction (v_readfirstlane, v_cmp ...)   5 wait states before a vector memory instruction reads it
    M0 written by a scalar instruction                                    1 before a load to LDS uses it
Every instruction is one wait state, s_nop n is n + 1.  Followed over all paths of every kernel; the parser itself is tested on a few lines."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2506_01084_amd import api

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
LINE = re.compile(r"^\t(\S+)\s*(.*?)\s*// ([0-9A-F]{12}): [0-9A-F ]+(?:<(.+?)(?:\+0x([0-9a-f]+))?>)?$")
VMEM = re.compile(r"(global|buffer|flat|scratch|tbuffer)_")


def _sgprs(operand):
    m = re.match(r"^s\[(\d+):(\d+)\]$", operand)
    if m:
        return [f"s{i}" for i in range(int(m[1]), int(m[2]) + 1)]
    if re.match(r"^s\d+$", operand) or operand in ("vcc_lo", "vcc_hi", "m0"):
        return [operand]
    return ["vcc_lo", "vcc_hi"] if operand == "vcc" else []


def _written(op, args):
    """SGPRs the instruction writes, and whether it is a vector instruction."""
    if op.startswith("v_"):
        if re.match(r"v_(readfirstlane|readlane|cmp)", op):
            return _sgprs(args[0]), True
        if re.match(r"v_(add|sub|subrev)c?_co|v_div_scale|v_mad_[iu]64", op):
            return _sgprs(args[1]), True
        return [], True
    if op.startswith("s_") and args and not re.match(r"s_(cmp|bitcmp|waitcnt|nop|cbranch|branch|barrier|sleep|setprio)", op):
        return _sgprs(args[0]), False
    return [], False


def short_waits(lines):
    """(address, instruction, register, wait states) of every memory instruction that comes too early in one kernel's listing."""
    code, at = [], {}
    for line in lines:
        m = LINE.match(line)
        if m:
            at[int(m[3], 16)] = len(code)
            code.append((m[1], [a.strip() for a in m[2].split(",")], int(m[3], 16), int(m[5], 16) if m[5] else (0 if m[4] else None)))
    if not code:
        return []
    base = code[0][2]
    state = [None] * len(code)           # register -> (wait states since it was written, those needed), the fewest over all paths
    state[0] = {}
    work, short = [0], {}
    while work:
        i = work.pop()
        op, args, addr, target = code[i]
        if VMEM.match(op):
            words = [w for a in args for w in a.split()]
            for reg in [r for w in words for r in _sgprs(w)] + (["m0"] if "lds" in words or "_lds_" in op else []):
                if reg in state[i]:
                    short[addr] = (hex(addr), " ".join([op, *args]), reg, state[i][reg][0])
        passed = int(args[0], 0) + 1 if op == "s_nop" else 1
        after = {r: (n + passed, need) for r, (n, need) in state[i].items() if n + passed < need}
        regs, vector = _written(op, args)
        for r in regs:
            after.pop(r, None)
            if vector:
                after[r] = (0, 5)
            elif r == "m0":
                after[r] = (0, 1)
        to = [] if op in ("s_endpgm", "s_branch", "s_setpc_b64") else [i + 1] if i + 1 < len(code) else []
        if op.startswith(("s_branch", "s_cbranch")):
            to.append(at[base + target])
        for j in to:
            merged = dict(state[j] or {})
            for r, v in after.items():
                merged[r] = min(merged.get(r, v), v)
            if state[j] is None or merged != state[j]:
                state[j] = merged
                work.append(j)
    return list(short.values())


def _listing(*instructions):
    return [f"\t{text:<60}// {4 * i:012X}: BF800000{tail}" for i, (text, tail) in enumerate(instructions)]


def test_the_reader_counts_wait_states_over_branches():
    late = [("v_readfirstlane_b32 s2, v0", ""), ("s_nop 2", ""), ("s_add_u32 m0, s9, 0", ""), ("s_nop 0", ""),
            ("buffer_load_dwordx4 v1, s[0:3], 0 offen lds", ""), ("s_endpgm", "")]
    assert short_waits(_listing(*late)) == []
    early = list(late)
    early[1] = ("s_nop 1", "")
    assert [s[2:] for s in short_waits(_listing(*early))] == [("s2", 4)]
    early[1], early[3] = late[1], ("s_cbranch_scc1 2", " <k+0x10>")
    assert short_waits(_listing(*early)) == []                     # the branch counts as one
    around = [("s_cbranch_scc1 2", " <k+0x8>"), ("s_branch 1", " <k+0xc>"), ("v_cmp_eq_u32_e64 s[6:7], v0, v1", ""),
              ("global_load_dwordx4 v[0:3], v4, s[6:7]", ""), ("s_endpgm", "")]
    assert [s[2:] for s in short_waits(_listing(*around))] in ([("s6", 0)], [("s7", 0)])
    m0 = [("s_mov_b32 m0, s3", ""), ("global_load_lds_dwordx4 v2, s[4:5]", ""), ("s_endpgm", "")]
    assert [s[2:] for s in short_waits(_listing(*m0))] == [("m0", 0)]


@pytest.mark.skipif(not os.path.exists(OBJDUMP), reason="no llvm-objdump")
def test_memory_instructions_wait_for_the_registers_they_read(tmp_path):
    lib = str(tmp_path / "libz2z.so")
    shutil.copy(api.LIB_PATH, lib)
    subprocess.run([OBJDUMP, "--offloading", lib], check=True, capture_output=True)       # (extracts next to the file)
    objects = sorted(p for p in tmp_path.iterdir() if "amdgcn" in p.name and "gfx950" in p.name)
    assert objects, "no gfx950 code in the library"
    short, kernels = [], 0
    for obj in objects:
        text = subprocess.run([OBJDUMP, "-d", str(obj)], check=True, capture_output=True, text=True).stdout
        for part in re.split(r"^[0-9a-f]{16} <(.+)>:$", text, flags=re.M)[2::2]:
            kernels += 1
            short += short_waits(part.split("\n"))
    assert kernels > 100, "kernels are missing from the listing"
    assert not short, short
