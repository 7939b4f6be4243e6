"""History ids are the caller's: counters, packed pairs, addresses.  The hash of the library's tables, compiled for the host, is
checked against chains that such ids could make; no GPU is involved."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_hash_of_ids_on_the_host(tmp_path):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not found")
    exe = str(tmp_path / "hash_check")
    cmd = [hipcc, "--cuda-host-only", "-std=c++17", "-O1", "-x", "hip",
           "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(ROOT, "paper_2007_11794_amd", "csrc"),
           os.path.join(ROOT, "tests", "host", "hash_check.cpp"), "-o", exe]
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout[-2000:] + r.stderr[-2000:]
