"""Builds the gfx950 shared library in-tree (hipcc cross-compiles without a GPU)."""
from __future__ import annotations

import glob
import os
import subprocess
import tempfile
from concurrent.futures import ThreadPoolExecutor

_HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(_HERE)
SRC = sorted(glob.glob(os.path.join(_HERE, "csrc", "*.hip")))
LIB = os.path.join(_HERE, "libsquant_hip.so")

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-fno-fast-math", "-ffp-contract=off", "-fhip-fp32-correctly-rounded-divide-sqrt",
    "-fno-gpu-flush-denormals-to-zero",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def build_hip(force: bool = True, extra=()) -> str:
    """One translation unit per kernel family, compiled side by side, and one link."""
    if force or not os.path.exists(LIB):
        hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
        jobs = int(os.environ.get("MAX_JOBS", 0)) or min(8, os.cpu_count() or 1)
        with tempfile.TemporaryDirectory() as tmp:
            def compile_one(src: str) -> str:
                obj = os.path.join(tmp, os.path.basename(src) + ".o")
                subprocess.check_call([hipcc, *HIPCC_FLAGS, *extra, "-I", os.path.join(ROOT, "include"),
                                       "-c", src, "-o", obj])
                return obj
            with ThreadPoolExecutor(jobs) as pool:
                objs = list(pool.map(compile_one, SRC))
            subprocess.check_call([hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", LIB])
    return LIB
