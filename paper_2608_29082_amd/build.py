"""Build the HIP library libmgl.so in-tree for gfx950.

    python -m paper_2608_29082_amd.build

Packed-FP32 instruction selection is disabled for every HIP translation unit
(some of its forms are not trusted on the target machines).
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(HERE, "libmgl.so")
ARCH = os.environ.get("MGL_OFFLOAD_ARCH", "gfx950")

HIP_FLAGS = [
    f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-result", "-Wno-unused-function",
]


def hipcc() -> str:
    for c in (os.environ.get("HIPCC"), shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if c and os.path.exists(c):
            return c
    raise RuntimeError("hipcc not found")


SOURCES = ("mgl.hip", "tail_f32.hip", "tail_f64.hip", "helm.hip", "hierarchy.cpp")


def build(verbose: bool = True) -> str:
    """Compile the sources of csrc/ side by side and link libmgl.so (always recompiles)."""
    tmp = LIB + ".tmp"
    objs = [f"{tmp}.{s.rsplit('.', 1)[0]}.o" for s in SOURCES]
    msgs = []

    def run(cmd):
        if verbose:
            print(" ".join(cmd), flush=True)
        res = subprocess.run(cmd, capture_output=True, text=True)
        # the host pass does not know the packed-fp32 feature; that warning is harmless
        out = [ln for ln in (res.stdout + res.stderr).splitlines() if "packed-fp32-ops" not in ln]
        if res.returncode != 0:
            raise RuntimeError("hipcc failed:\n" + "\n".join(out))
        msgs.extend(out)

    def compile_one(k):
        run([hipcc(), *HIP_FLAGS, f"-I{INCLUDE}", f"-I{CSRC}", "-c", os.path.join(CSRC, SOURCES[k]), "-o", objs[k]])

    try:
        with ThreadPoolExecutor(len(SOURCES)) as pool:
            list(pool.map(compile_one, range(len(SOURCES))))
        run([hipcc(), f"--offload-arch={ARCH}", "-shared", *objs, "-o", tmp])
    finally:
        for o in objs:
            if os.path.exists(o):
                os.remove(o)
    if verbose and msgs:
        print("\n".join(msgs), file=sys.stderr)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    build()
