"""The weight-streaming form of the output projection awaits the hidden block with a count of younger loads: in the compiled
code of every kernel that contains it, at least that many loads of the wave must lie between the last direct-to-LDS load and
the wait (hipcc cross-compiles without a GPU)."""
import os
import re
import subprocess

import pytest

from paper_2007_11794_amd import build as b


def loads_before_waits(lines):
    """Per wait for the hidden block: loads to registers since the last direct-to-LDS load in front of it."""
    out, n, seen = [], 0, False
    for line in lines:
        s = line.strip()
        if re.match(r"_Z\S+:", line):
            n, seen = 0, False
        if s.startswith("global_load_lds"):
            n, seen = 0, True
        elif s.startswith("global_load"):
            n += 1
        elif seen and re.match(r"s_waitcnt vmcnt\(12\) ; hidden block$", s):
            out.append(n)
    return out


def test_the_scan_counts():
    asm = ["_Zk:", "global_load_lds_dwordx4 v1, s[0:1]", "global_load_dwordx4 v[4:7], v[0:1], off", "s_waitcnt vmcnt(12)",
           "s_waitcnt vmcnt(12) ; hidden block"]
    assert loads_before_waits(asm) == [1]


# source, waits in it: one per instance of the streaming form
@pytest.mark.parametrize("source,waits", [("outproj_stream.hip", 12), ("outproj_staged.hip", 72), ("outproj_tiled.hip", 8),
                                          ("outproj_rowstream.hip", 2), ("outproj_split2.hip", 12)])
def test_enough_younger_loads(source, waits, tmp_path):
    out = str(tmp_path / "kernel.s")
    subprocess.run([b._hipcc()] + b.flags_of(source) + ["-S", "--cuda-device-only", os.path.join(b.CSRC, source), "-o", out], check=True,
                   capture_output=True)
    with open(out) as f:
        counts = loads_before_waits(f.read().splitlines())
    assert len(counts) >= waits and min(counts) >= 12, counts
