"""Loads the compiler does not see as loads (inline assembly with an output operand, awaited by hand): in the compiled
code nothing may touch such a register between the load and the wait that covers it.  Checked on the assembly of the
kernels that use them (hipcc cross-compiles without a GPU)."""
import os
import re
import subprocess

import pytest

from paper_2007_11794_amd import build as b


def registers(text):
    out = {int(r) for r in re.findall(r"\bv(\d+)\b", text)}
    for lo, hi in re.findall(r"\bv\[(\d+):(\d+)\]", text):
        out |= set(range(int(lo), int(hi) + 1))
    return out


def violations(lines):
    """Instructions that name the destination of an inline-assembly load which may still be in flight.  Vector memory
    operations complete in order, so `vmcnt(n)` retires all but the n youngest; straight-line scan per function."""
    flying, in_asm, found = [], False, []
    for line in lines:
        s = line.strip()
        if s.startswith(";"):
            in_asm = "ASMSTART" in s or (in_asm and "ASMEND" not in s)
            continue
        if re.match(r"_Z\S+:", line):
            flying = []
        if not s or s.startswith("."):
            continue
        op, _, rest = s.split(";")[0].strip().partition(" ")
        if op == "s_waitcnt":
            n = re.search(r"vmcnt\((\d+)\)", rest)
            if n:
                flying = flying[max(0, len(flying) - int(n.group(1))):]
            continue
        loads = op.startswith(("global_load", "buffer_load", "scratch_load"))
        target, _, sources = rest.partition(",")
        to_registers = loads and "lds" not in op
        named = registers(sources if to_registers and in_asm else rest)
        if any(named & f for f in flying):
            found.append(s)
        if loads or op.startswith(("global_store", "global_atomic")):
            flying.append(registers(target) if to_registers and in_asm else set())
    return found


def test_the_scan_finds_a_read_in_front_of_the_wait():
    asm = ["_Zk:", ";APP ASMSTART", "global_load_dwordx4 v[4:7], v[0:1], off", ";ASMEND", "v_mov_b32_e32 v9, v6",
           "s_waitcnt vmcnt(0)", "v_mov_b32_e32 v10, v6"]
    assert violations(asm) == ["v_mov_b32_e32 v9, v6"]


@pytest.mark.parametrize("source", ["outproj_rowstream.hip", "outproj_staged.hip"])
def test_operands_stay_untouched_until_they_have_landed(source, tmp_path):
    out = str(tmp_path / "kernel.s")
    subprocess.run([b._hipcc()] + b.flags_of(source) + ["-S", "--cuda-device-only", os.path.join(b.CSRC, source), "-o", out], check=True,
                   capture_output=True)
    with open(out) as f:
        lines = f.read().splitlines()
    assert any("ASMSTART" in x for x in lines)
    assert violations(lines) == []
