"""Builds libpre3.so (HIP kernels + C ABI) for gfx950 with hipcc, in-tree."""
from __future__ import annotations

import os
import subprocess
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OBJ = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "libpre3.so")
SOURCES = ["grammar.cpp", "lr1.cpp", "tables.cpp", "token_edges.cpp", "symbol_edges.cpp", "api.cpp",
           "mask_kernels.hip", "apply_kernels.hip", "sampler_kernels.hip", "advance_kernels.hip"]
# The first 14 words of a kernel's arguments arrive in scalar registers with the launch, where they are plain pointers and
# sizes (a struct ends the sequence: kernels that take the tables by value take them behind these): what reads an input or
# the tables' copy in device memory does not wait for the argument segment first.  (jump-forward asks for its inputs at
# once; the advancing kernels and the mask kernel still ask for the table pointers before.)  Bursts of 8 steps: fill, mask
# and advance of 96 x 100,003 as three calls 173.8 -> 168.0 us, jump-forward with 128 x 128,256 208.9 -> 202.5,
# 2,048 x 128,256 1,464 -> 1,446.
FLAGS = ["-O3", "--offload-arch=gfx950", "-std=c++17", "-fPIC", "-pthread",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-mllvm", "-amdgpu-kernarg-preload-count=14"]
# the host pass does not know the packed-fp32 target feature and says so: harmless
_NOISE = "is not a recognized feature for this target"


def _run(cmd):
    proc = subprocess.run(cmd, capture_output=True, text=True)
    err = "\n".join(l for l in proc.stderr.splitlines() if _NOISE not in l)
    if proc.returncode != 0:
        raise RuntimeError("hipcc failed: " + " ".join(cmd[-3:]) + "\n" + err)
    return err


def _newest_header() -> float:
    paths = [os.path.join(CSRC, f) for f in os.listdir(CSRC) if f.endswith((".hpp", ".h"))]
    paths.append(os.path.join(HERE, "..", "include", "pre3.h"))
    return max(os.path.getmtime(p) for p in paths)


def build(verbose: bool = False, incremental: bool = False) -> str:
    """Compiles every source to an object (in parallel) and links the shared library.  With
    `incremental` an object newer than its source and every header, and built with the same flags, is kept."""
    os.makedirs(OBJ, exist_ok=True)
    newest_h = _newest_header()
    built_with = os.path.join(OBJ, "flags")              # of the objects that lie there
    flags = " ".join(FLAGS)
    if os.path.exists(built_with):
        with open(built_with) as f:
            incremental = incremental and f.read() == flags
        os.remove(built_with)                            # until all of them are built
    else:
        incremental = False
    jobs = []
    for s in SOURCES:
        src, obj = os.path.join(CSRC, s), os.path.join(OBJ, s + ".o")
        fresh = os.path.exists(obj) and os.path.getmtime(obj) > max(os.path.getmtime(src), newest_h)
        if not (incremental and fresh):
            jobs.append(["hipcc", *FLAGS, "-c", "-o", obj, src])
    with ThreadPoolExecutor(max_workers=min(8, os.cpu_count() or 1)) as pool:
        notes = list(pool.map(_run, jobs))
    with open(built_with, "w") as f:
        f.write(flags)
    notes.append(_run(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", "-pthread", "-o", LIB,
                       *[os.path.join(OBJ, s + ".o") for s in SOURCES]]))
    if verbose:
        print("\n".join(n for n in notes if n.strip()))
    return LIB


if __name__ == "__main__":
    import sys
    print(build(verbose=True, incremental="--incremental" in sys.argv))
