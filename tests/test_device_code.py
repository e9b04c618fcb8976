"""The built kernels hold no vector instruction where no lane is active.

A loop that lanes leave one by one ends with EXEC empty.  When registers are
short the compiler can place a spill between that exit and the instruction
that restores EXEC: it then stores nothing, and what is reloaded later is
whatever the stack held.  The march kernels met this once; the disassembly of
the built library is searched for it."""

import os
import re
import shutil
import subprocess

import pytest

from paper_1909_05423_amd import _lib

OBJDUMP = shutil.which("llvm-objdump", path=os.pathsep.join(
    [os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "llvm", "bin"), os.environ.get("PATH", "")]))

_VECTOR = re.compile(r"(v_(?!readlane|writelane|readfirstlane|nop)|ds_(?!nop)|global_|scratch_|buffer_|flat_)")
_EXEC = re.compile(r"(s_\w+ exec[, _]|s_\w+saveexec|v_cmpx)")
_LINE = re.compile(r"^\s+(\S.*?)\s*// ([0-9A-F]+):")
_TARGET = re.compile(r"^s_c?branch\w* (\d+)")


def inactive_vector_instructions(lines):
    """Vector instructions that only run with EXEC empty: after a branch that is
    taken while any lane is active, up to the next write of EXEC or the next
    place that is also reached from elsewhere."""
    code, targets = [], set()
    for line in lines:
        m = _LINE.match(line)
        if not m:
            code.append(None)   # a kernel's label
            continue
        text, addr = m.group(1), int(m.group(2), 16)
        code.append((addr, text))
        t = _TARGET.match(text)
        if t:
            off = int(t.group(1))
            targets.add(addr + 4 + 4 * (off - 65536 if off >= 32768 else off))
    found, empty = [], False
    for item in code:
        if item is None:
            empty = False
            continue
        addr, text = item
        if addr in targets or _EXEC.match(text) or text.startswith(("s_branch", "s_endpgm", "s_setpc")):
            empty = False
        elif empty and _VECTOR.match(text):
            found.append((hex(addr), text))
        if text.startswith("s_cbranch_execnz"):
            empty = True
    return found


def test_search_finds_a_lost_store():
    loop = ["\ts_andn2_b64 exec, exec, s[0:1]  // 000000000100: 0",
            "\ts_cbranch_execnz 65534  // 000000000104: 0",
            "\tv_writelane_b32 v255, s29, 17  // 000000000108: 0",
            "\tscratch_store_dwordx2 off, v[232:233], off offset:316  // 000000000110: 0",
            "\ts_or_b64 exec, exec, s[0:1]  // 000000000118: 0",
            "\tv_mov_b32_e32 v0, 0  // 00000000011C: 0"]
    assert inactive_vector_instructions(loop) == [("0x110", "scratch_store_dwordx2 off, v[232:233], off offset:316")]
    # the same place reached from elsewhere too, or with EXEC restored first
    assert inactive_vector_instructions(["\ts_cbranch_scc1 3  // 0000000000FC: 0"] + loop[:2] + loop[3:]) != []
    assert inactive_vector_instructions(["\ts_cbranch_scc1 4  // 0000000000FC: 0"] + loop) == []
    assert inactive_vector_instructions(loop[:2] + [loop[4], loop[3]]) == []


@pytest.mark.skipif(OBJDUMP is None, reason="llvm-objdump not found")
def test_no_vector_instruction_runs_without_lanes(tmp_path):
    lib = tmp_path / "lib.so"
    shutil.copyfile(_lib.LIB_PATH, lib)
    subprocess.run([OBJDUMP, "--offloading", str(lib)], check=True, stdout=subprocess.DEVNULL, cwd=tmp_path)
    objects = sorted(p for p in tmp_path.iterdir() if p.name.endswith("gfx950"))
    assert objects
    kernels, found = 0, []
    for p in objects:
        dis = subprocess.run([OBJDUMP, "-d", "--no-show-raw-insn", str(p)], check=True, stdout=subprocess.PIPE,
                             text=True).stdout.splitlines()
        kernels += sum(line.endswith(">:") for line in dis)
        found += inactive_vector_instructions(dis)
    assert kernels > 100
    assert not found, found[:10]
