"""Manually inserted wait states of the gfx950 vector ALU in the compiled kernels.

A result that one vector instruction leaves for another may not be read at
once in three cases, and the hardware does not wait by itself:
  - a scalar register or vcc written by the vector ALU, read by it again: two
    wait states in between;
  - a vector register read through DPP: two;
  - a vector register read by v_readlane or v_readfirstlane: one.
The compiler keeps to this for its own instructions and not inside an inline
asm block, so every kernel with inline asm is compiled to assembly here and
read. An instruction is one wait state, s_nop N is N + 1.
"""
import os
import re
import subprocess

import pytest

from paper_1501_01405_amd import _build

DST2 = re.compile(r"v_(mad_u64|mad_i64|div_scale|(add|sub|subrev|addc|subb|subbrev)_co_)")
MODIFIERS = re.compile(r"\s(row_|quad_perm|wave_|bank_|bound_|op_sel|src0_sel|src1_sel|dst_|neg_|mul:|clamp).*")


def registers(operand):
    o = re.sub(r"^-|^abs\(|[|)]", "", operand.strip())
    if o == "vcc":
        return {("s", "vcc")}
    m = re.fullmatch(r"([vsa])(\d+)", o)
    if m:
        return {(m.group(1), int(m.group(2)))}
    m = re.fullmatch(r"([vsa])\[(\d+):(\d+)\]", o)
    return {(m.group(1), i) for i in range(int(m.group(2)), int(m.group(3)) + 1)} if m else set()


def union(operands):
    return set().union(set(), *(registers(o) for o in operands))


def early_reads(lines):
    """(line number, line) of every read that comes too early after its write."""
    found, recent = [], []  # recent: (wait states, registers written, by the vector ALU)
    for number, line in enumerate(lines, 1):
        m = re.match(r"\t([vsdg]\w+)\s*([^;]*)", line)
        if not m:
            continue
        name, body = m.groups()
        if name == "s_nop":
            recent.append((int(body) + 1, set(), False))
            continue
        vector = name.startswith("v_")
        dpp = bool(re.search(r"\b(row_\w+|quad_perm|wave_\w+):", body)) or "_dpp" in name
        operands = MODIFIERS.sub("", body).split(",")
        n_dst = 2 if DST2.match(name) else 1
        written, read = union(operands[:n_dst]), union(operands[n_dst:])
        if vector:
            need = {r: 2 for r in read if r[0] == "s"}
            if dpp:
                need.update({r: 2 for r in registers(operands[n_dst])})
            if name.startswith(("v_readlane", "v_readfirstlane")):
                need.update({r: 1 for r in registers(operands[1])})
            passed, settled = 0, set()
            for states, regs, by_vector in reversed(recent):
                if any(r in regs and r not in settled and passed < n for r, n in need.items()
                       ) and by_vector:
                    found.append((number, line.strip()))
                settled |= regs
                passed += states
        recent = (recent + [(1, written, vector)])[-4:]
    return found


def test_the_reader_finds_early_reads():
    code = ["\tv_sub_co_u32 v1, vcc, v2, v3", "\tv_addc_co_u32 v4, vcc, v4, v4, vcc",      # early
            "\ts_nop 1", "\tv_cndmask_b32_e32 v5, v6, v7, vcc",                            # two passed
            "\tv_cmp_lt_u32_e64 s[2:3], v1, v2", "\tv_mov_b32 v9, v8", "\ts_nop 0",
            "\tv_cndmask_b32_e64 v5, v6, v7, s[2:3]",                                      # in time
            "\tv_add_f32 v1, v2, v3", "\tv_mov_b32 v9, v8",
            "\tv_mov_b32_dpp v4, v1 row_shr:1 row_mask:0xf bank_mask:0xf",                 # early
            "\tv_min_f32 v6, v2, v3", "\tv_readlane_b32 s4, v6, 63",                       # early
            "\ts_lshl_b32 s4, s5, 2", "\tv_add_u32 v1, s4, v2"]                            # scalar write
    assert [n for n, _ in early_reads(code)] == [2, 11, 13]


@pytest.mark.parametrize("source", ["ff", "mm1", "pi"])
def test_no_vector_result_is_read_too_early(source, tmp_path):
    src = os.path.join(_build.CSRC, source + ".hip")
    out = str(tmp_path / (source + ".s"))
    flags = [f for f in _build.FLAGS if f not in ("-shared", "-fPIC")]
    subprocess.run([_build.HIPCC, *flags, "-S", "--cuda-device-only", src, "-o", out], check=True,
                   stderr=subprocess.DEVNULL)
    with open(out) as f:
        lines = f.read().splitlines()
    assert sum("v_" in ln for ln in lines) > 1000
    found = early_reads(lines)
    assert not found, found[:5]
