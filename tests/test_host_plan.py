"""The work split of the output projection is planned by one small function that the host (launch
sizes) and the kernels (with the row count they read on the device) both evaluate; the kernel that
merges the partials afterwards derives the number of partials from it again.  This test compiles
that function for the host and checks its properties; no GPU is involved."""
import os
import shutil
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def check_on_the_host(tmp_path, name, libraries=()):
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not found")
    exe = str(tmp_path / name)
    cmd = [hipcc, "--cuda-host-only", "-std=c++17", "-O1", "-x", "hip",
           "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(ROOT, "paper_2007_11794_amd", "csrc"),
           os.path.join(ROOT, "tests", "host", name + ".cpp"), "-o", exe, "-x", "none"] + list(libraries)
    r = subprocess.run(cmd, capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-2000:]
    r = subprocess.run([exe], capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and r.stdout.strip() == "ok", r.stdout[-2000:] + r.stderr[-2000:]


def test_work_split_arithmetic_on_the_host(tmp_path):
    check_on_the_host(tmp_path, "plan_check")


@pytest.mark.parametrize("name", ["ahead_check",      # weights read ahead in the order of their reader
                                  "whole_check"])     # launches and kernels of the hidden update's whole form
def test_dispatch_of_the_built_library(tmp_path, name):
    import paper_2007_11794_amd as rn
    rn.lib()                                   # (there, or it says so)
    check_on_the_host(tmp_path, name, [rn.lib_path(), "-Wl,-rpath," + os.path.dirname(rn.lib_path())])
