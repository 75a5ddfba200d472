"""Compile the HIP library for gfx950 in-tree (hipcc cross-compiles without a GPU)."""
from __future__ import annotations

import os
import subprocess
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libfb_amd.so")
SOURCES = ["fb_kernels.hip", "fb_graph.cpp", "fb_sell.cpp", "fb_stream.cpp", "fb_pstream.cpp", "fb_small.cpp", "fb_api.cpp", "fb_leaky.hip",
           "fb_small.hip", "fb_small_linear.hip", "fb_post_small.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "-O3", "-std=c++17", "-fPIC", "--offload-arch=gfx950",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",   # never emit packed FP32 arithmetic
    "-Wall", "-Wno-unused-function", "-x", "hip",
]


def sources():
    return [os.path.join(CSRC, s) for s in SOURCES]


def is_stale() -> bool:
    if not os.path.exists(LIB):
        return True
    t = os.path.getmtime(LIB)
    deps = sources() + [os.path.join(CSRC, h) for h in ("fb_internal.h", "fb_device.h", "fb_small_run.h")] + [os.path.join(HERE, "..", "include", "fb.h")]
    return any(os.path.getmtime(d) > t for d in deps)


def build_library(verbose: bool = False) -> str:
    # one compiler per source, side by side, then the link
    objs, running = [], []
    for src in sources():
        obj = os.path.join(tempfile.gettempdir(), f"fb_amd_{os.getpid()}_{os.path.basename(src)}.o")
        cmd = [HIPCC] + FLAGS + ["-c", src, "-o", obj]
        if verbose:
            print(" ".join(cmd))
        objs.append(obj)
        running.append(subprocess.Popen(cmd))
    codes = [p.wait() for p in running]
    try:
        if any(codes):
            raise subprocess.CalledProcessError(next(c for c in codes if c), "hipcc")
        subprocess.check_call([HIPCC, "-shared", "--offload-arch=gfx950"] + objs + ["-o", LIB])
    finally:
        for obj in objs:
            if os.path.exists(obj):
                os.remove(obj)
    return LIB


if __name__ == "__main__":
    print(build_library(verbose=True))
