"""Compiled-code check of libgcdf.so (no GPU): no register is spilled to scratch memory
at a join of divergent control flow before the join restores EXEC.

Such a store keeps the value of the lanes that came through the branch only; a reload
after the join gives every other lane whatever the slot held.  The compiler has placed
one there: in a serving kernel whose tile prologue runs in one wave, the other waves
reloaded the address of their rows of J, and the stores through it faulted."""
import os
import re
import shutil
import subprocess

import pytest

from paper_2601_18548_amd import build

OBJDUMP = "/opt/rocm/llvm/bin/llvm-objdump"
INS = re.compile(r"^\t(\S+)(.*?)//\s*([0-9A-F]+):.*?(?:<\S+\+0x([0-9a-f]+)>|<\S+>)?$")


def functions(text):
    """(name, [(offset, instruction, branch target's offset or None)]) of a disassembly."""
    name, base, out = None, 0, []
    for line in text.splitlines():
        m = re.match(r"^([0-9a-f]+) <(\S+)>:", line)
        if m:
            if out:
                yield name, out
            base, name, out = int(m[1], 16), m[2], []
            continue
        m = INS.match(line)
        if m:
            target = int(m[4], 16) if m[4] and "branch" in m[1] else None
            out.append((int(m[3], 16) - base, (m[1] + m[2]).strip(), target))
    if out:
        yield name, out


def spills_ahead_of_exec_restore(code):
    """scratch stores that precede `s_or_b64 exec, exec, ...` in the same basic block."""
    starts = {t for _, _, t in code if t is not None}
    found, block = [], []
    for off, ins, target in code:
        if off in starts:
            block = []
        if ins.startswith("scratch_store"):
            block.append("%x: %s" % (off, ins))
        if re.match(r"s_or_b64 exec, exec\b", ins):
            found += block
        if target is not None or re.match(r"s_\w+ exec\b|s_\w+saveexec|v_cmpx", ins):
            block = []
    return found


def test_the_check_sees_a_spill_at_a_join():
    text = "\n".join([
        "0000000000001000 <k>:",
        "\ts_mov_b64 exec, s[0:1]                 // 000000001000: BEFE0100",
        "\ts_cbranch_execz 1                      // 000000001004: BF880001 <k+0xc>",
        "\tv_mov_b32_e32 v0, 0                    // 000000001008: 7E000280",
        "\tscratch_store_dwordx2 off, v[2:3], off offset:8 // 00000000100C: DC740008",
        "\ts_or_b64 exec, exec, s[4:5]            // 000000001014: 87FE047E",
    ])
    (name, code), = functions(text)
    assert name == "k" and spills_ahead_of_exec_restore(code) == ["c: scratch_store_dwordx2 off, v[2:3], off offset:8"]
    moved = [code[0], code[1], code[2], (12, code[4][1], None), (20, code[3][1], None)]
    assert spills_ahead_of_exec_restore(moved) == []


def test_no_spill_ahead_of_an_exec_restore(tmp_path):
    if not os.path.exists(OBJDUMP):
        pytest.skip("no llvm-objdump")
    shutil.copy(build.LIB, tmp_path / "lib.so")
    subprocess.check_call([OBJDUMP, "--offloading", "lib.so"], cwd=tmp_path, stdout=subprocess.DEVNULL)
    kernels, bad = 0, []
    for f in sorted(tmp_path.glob("lib.so.*gfx950")):
        text = subprocess.run([OBJDUMP, "-d", "--mcpu=gfx950", str(f)], check=True, capture_output=True, text=True).stdout
        for name, code in functions(text):
            kernels += 1
            bad += ["%s %s" % (name, x) for x in spills_ahead_of_exec_restore(code)]
    assert kernels > 50 and not bad, "\n".join(bad)
