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


def instructions(lines):
    """Per function: its instructions as (operation, rest, within inline assembly), and the index that each label stands for."""
    functions, in_asm = [], False
    for line in lines:
        s = line.strip()
        if s.startswith(";"):
            in_asm = "ASMSTART" in s or (in_asm and "ASMEND" not in s)
            continue
        if re.match(r"_Z\S+:", line):
            functions.append(([], {}))
        label = re.match(r"(\.L\w+):", s)
        if label:
            functions[-1][1][label.group(1)] = len(functions[-1][0])
        if not functions or not s or s.startswith(".") or s.endswith(":"):
            continue
        op, _, rest = s.split(";")[0].strip().partition(" ")
        functions[-1][0].append((op, rest.strip(), in_asm))
    return functions


def violations(lines):
    """Instructions that name the destination of an inline-assembly load which may still be in flight.  Vector memory
    operations complete in order, so `vmcnt(n)` retires all but the n youngest (63 at most are in flight).  Every way through
    a function is followed, loops included: a branch takes the list of what is in flight to its target, once per list."""
    found = []
    for code, labels in instructions(lines):
        ways, seen = [(0, ())], set()
        while ways:
            at, flying = ways.pop()
            while at < len(code):
                op, rest, in_asm = code[at]
                if op == "s_waitcnt":
                    n = re.search(r"vmcnt\((\d+)\)", rest)
                    if n:
                        flying = flying[max(0, len(flying) - int(n.group(1))):]
                elif op.startswith(("s_branch", "s_cbranch")):
                    while flying and not flying[0]:
                        flying = flying[1:]
                    to = labels.get(rest)
                    if to is not None and (to, flying) not in seen:
                        seen.add((to, flying))
                        ways.append((to, flying))
                    if op == "s_branch" or (at + 1, flying) in seen:
                        break
                    seen.add((at + 1, flying))
                elif op == "s_endpgm":
                    break
                else:
                    loads = op.startswith(("global_load", "buffer_load", "scratch_load"))
                    target, _, sources = rest.partition(",")
                    to_registers = loads and "lds" not in op
                    named = registers(sources if to_registers and in_asm else rest)
                    if any(named & f for f in flying) and "%s %s" % (op, rest) not in found:
                        found.append("%s %s" % (op, rest))
                    if loads or op.startswith(("global_store", "global_atomic")):
                        flying = (flying + (frozenset(registers(target) if to_registers and in_asm else ()),))[-63:]
                at += 1
    return found


def test_the_scan_finds_a_read_in_front_of_the_wait():
    asm = ["_Zk:", ";APP ASMSTART", "global_load_dwordx4 v[4:7], v[0:1], off", ";ASMEND", "v_mov_b32_e32 v9, v6",
           "s_waitcnt vmcnt(0)", "v_mov_b32_e32 v10, v6"]
    assert violations(asm) == ["v_mov_b32_e32 v9, v6"]


def test_the_scan_follows_loops_and_branches():
    load = [";APP ASMSTART", "global_load_dwordx4 v[4:7], v[0:1], off", ";ASMEND"]
    # the load at a loop's end is read at its head, in front of the wait there
    asm = ["_Zk:", ".LBB0_1:", "v_mov_b32_e32 v9, v6", "s_waitcnt vmcnt(0)"] + load + ["s_cbranch_scc1 .LBB0_1", "s_endpgm"]
    assert violations(asm) == ["v_mov_b32_e32 v9, v6"]
    # a branch leads around the wait
    asm = ["_Zk:"] + load + ["s_cbranch_scc1 .LBB0_1", "s_waitcnt vmcnt(0)", ".LBB0_1:", "v_mov_b32_e32 v9, v6", "s_endpgm"]
    assert violations(asm) == ["v_mov_b32_e32 v9, v6"]
    asm = ["_Zk:"] + load + ["s_cbranch_scc1 .LBB0_1", ".LBB0_1:", "s_waitcnt vmcnt(0)", "v_mov_b32_e32 v9, v6", "s_endpgm"]
    assert violations(asm) == []


@pytest.mark.parametrize("source", ["outproj_rowstream.hip", "outproj_staged.hip"])
def test_operands_stay_untouched_until_they_have_landed(source, tmp_path):
    out = str(tmp_path / "kernel.s")
    subprocess.run([b._hipcc()] + b.flags_of(source) + ["-S", "--cuda-device-only", os.path.join(b.CSRC, source), "-o", out], check=True,
                   capture_output=True)
    with open(out) as f:
        lines = f.read().splitlines()
    assert any("ASMSTART" in x for x in lines)
    assert violations(lines) == []
