"""Builds libhxt.so (HIP, gfx950) in-tree with hipcc.  No GPU is needed to compile."""
from __future__ import annotations

import os
import subprocess
import tempfile
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
LIB = os.path.join(PKG, "libhxt.so")
SOURCES = [os.path.join(PKG, "csrc", f) for f in ("hxt_device.hip", "hxt_transpose.hip", "hxt_transpose_span.hip", "hxt_message_pack.hip",
                                                      "hxt_message_unpack.hip", "hxt_plan.cpp")]
HEADERS = [os.path.join(PKG, "csrc", f) for f in ("hxt_internal.h", "hxt_kernels.h", "hxt_launch.h", "hxt_rules.h")] + \
          [os.path.join(ROOT, "include", "hxt.h")]


def hipcc() -> str:
    for cand in (os.environ.get("HIPCC"), "/opt/rocm/bin/hipcc", "hipcc"):
        if cand and (os.path.sep not in cand or os.path.exists(cand)):
            return cand
    raise RuntimeError("hipcc not found")


FLAGS = ["-O3", "-std=c++20", "-fPIC", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wextra", "-Wno-unused-parameter",
         "-I", os.path.join(ROOT, "include"), "-I", os.path.join(PKG, "csrc")]


def compile_one(src: str, obj: str) -> None:
    subprocess.run([hipcc(), "--offload-arch=gfx950", *FLAGS, "-c", "-o", obj, src], check=True)


def stale() -> bool:
    if not os.path.exists(LIB):
        return True
    t = os.path.getmtime(LIB)
    return any(os.path.getmtime(f) > t for f in SOURCES + HEADERS)


def build(force: bool = True) -> str:
    if force or stale():
        with tempfile.TemporaryDirectory() as tmp, ThreadPoolExecutor(len(SOURCES)) as pool:
            objs = [os.path.join(tmp, os.path.basename(s) + ".o") for s in SOURCES]
            list(pool.map(compile_one, SOURCES, objs))
            subprocess.run([hipcc(), "--offload-arch=gfx950", "-shared", "-o", LIB, *objs], check=True)
    return LIB


if __name__ == "__main__":
    print(build())
