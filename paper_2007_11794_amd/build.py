"""Build librnnlm.so (HIP, gfx950 only) in-tree with hipcc.

    python -m paper_2007_11794_amd.build            # rebuild what changed
    python -m paper_2007_11794_amd.build --force    # rebuild everything
"""
from __future__ import annotations

import concurrent.futures
import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "librnnlm.so")
SOURCES = ["api.hip", "dedup.hip", "recur.hip", "recur_whole.hip", "outproj.hip", "outproj_staged.hip", "outproj_tiled.hip", "outproj_stream.hip", "outproj_rowstream.hip", "outproj_split2.hip", "query.hip", "step_few.hip",
           "load_kernels.hip", "cache.hip", "index_table.hip", "hs.hip", "diag.hip"]
HEADERS = [os.path.join(CSRC, "rnnlm_internal.h"), os.path.join(CSRC, "device_utils.h"),
           os.path.join(CSRC, "outproj_stream_body.h"), os.path.join(CSRC, "dedup_small_body.h"), os.path.join(CSRC, "recur_math.h"),
           os.path.join(CSRC, "recur_parts.h"), os.path.join(CSRC, "recur_whole.h"),
           os.path.join(ROOT, "include", "rnnlm.h"), os.path.join(ROOT, "include", "rnnlm_diag.h")]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fno-gpu-rdc",
         # packed-fp32 instructions stay off: the compiler must not form them on its own
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-function",
         "-I" + os.path.join(ROOT, "include"), "-I" + CSRC]

# These kernels' loops begin at a fetch line.  Staged: V = 60000, H = 128, 4096 rows 60.3 against 59.6 us.  Two-term: left where they fall, the same instructions took 158 to 173 us (V = 65536,
# H = 512, fp32, 1024 rows) and 32.6 to 34.3 (V = 8000, H = 1200, 40 rows), depending on what stands in front of them.
# Streaming: V = 1000000, H = 128, 10 rows 39.3 against 38.5 us.
# Staged: sums of matrix products stay in VGPRs in the kernels that may use 512 registers; in AGPRs each was copied out and
# back (fp32, 64 rows known on the device only: V = 65536, H = 512 27.2 against 26.0 us, V = 50000, H = 384, 50 rows 19.0 against 17.2).
FILE_FLAGS = {"outproj_stream.hip": ["-falign-loops=64"], "outproj_split2.hip": ["-falign-loops=64"], "outproj_staged.hip": ["-falign-loops=64", "-mllvm", "-amdgpu-mfma-vgpr-form=1"]}


def flags_of(src: str) -> list:
    return FLAGS + FILE_FLAGS.get(src, [])


def _hipcc() -> str:
    for c in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if c and (os.path.isabs(c) and os.path.exists(c) or not os.path.isabs(c)):
            return c
    return "hipcc"


def _stale(target: str, deps) -> bool:
    if not os.path.exists(target):
        return True
    t = os.path.getmtime(target)
    return any(os.path.getmtime(d) > t for d in deps)


def _compile(src: str, force: bool, extra) -> str:
    obj = os.path.join(OBJ, os.path.splitext(src)[0] + ".o")
    path = os.path.join(CSRC, src)
    if force or _stale(obj, [path] + HEADERS):
        cmd = [_hipcc()] + flags_of(src) + list(extra) + ["-c", path, "-o", obj]
        r = subprocess.run(cmd, capture_output=True, text=True)
        err = "\n".join(l for l in r.stderr.splitlines()
                        if "packed-fp32-ops" not in l)      # the host pass does not know the feature
        if r.returncode != 0:
            raise RuntimeError("hipcc failed for %s:\n%s" % (src, err))
        if err.strip():
            sys.stderr.write(err + "\n")
    return obj


def build(force: bool = False, extra_flags=()) -> str:
    os.makedirs(OBJ, exist_ok=True)
    with concurrent.futures.ThreadPoolExecutor(max_workers=min(8, len(SOURCES))) as ex:
        objs = list(ex.map(lambda s: _compile(s, force, extra_flags), SOURCES))
    if force or _stale(LIB, objs):
        tmp = LIB + ".tmp.%d" % os.getpid()
        subprocess.check_call([_hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs)
        os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(force="--force" in sys.argv))
