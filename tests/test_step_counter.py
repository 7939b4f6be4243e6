"""The one-launch step finds its last workgroup with a count in the handle's scratch, which must be zero again behind every
launch, whatever overlapped it.  The count's rule on the CPU, and that the compiled kernels count by this rule and
nothing else (hipcc cross-compiles without a GPU)."""
import os
import random
import re
import subprocess

from paper_2007_11794_amd import build as b


def wrapping(count, S):
    """atomicInc(count, S - 1): the value found, the value left."""
    return count, 0 if count >= S - 1 else count + 1


def test_the_count_is_zero_behind_launches_that_overlapped():
    rng = random.Random(3)
    for S in (1, 2, 40, 160):
        for launches in (1, 2, 3):
            arrivals, count, last = [i for i in range(launches) for _ in range(S)], 0, 0
            rng.shuffle(arrivals)
            for _ in arrivals:
                found, count = wrapping(count, S)
                last += found == S - 1
            assert count == 0 and last == launches


def counting(lines):
    """Operations on memory, by kernel, that read and write at once."""
    out, name = {}, None
    for line in lines:
        label = re.match(r"(_Z\S+):", line)
        name = label.group(1) if label else name
        op = re.match(r"\s+((?:global|flat|buffer)_atomic_\w+)", line)
        if op:
            out.setdefault(name, set()).add(op.group(1))
    return out


def test_the_kernels_count_by_that_rule(tmp_path):
    out = str(tmp_path / "kernel.s")
    subprocess.run([b._hipcc()] + b.flags_of("step_few.hip") + ["-S", "--cuda-device-only", os.path.join(b.CSRC, "step_few.hip"), "-o", out],
                   check=True, capture_output=True)
    with open(out) as f:
        kernels = {k: ops for k, ops in counting(f.read().splitlines()).items() if "step_few_kernel" in k}
    assert len(kernels) == 4                                       # two types, two forms of the log-sum-exp
    for ops in kernels.values():
        assert ops == {"global_atomic_inc", "global_atomic_or"}, ops        # the count, the flags
