"""Builds ``libadasum.so`` (gfx950) in-tree with hipcc.

Usage: ``python -m paper_2006_02924_amd.build``.  hipcc cross-compiles without a
GPU.  The library is written next to this file so that it travels with the
source tree.
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB_PATH = os.path.join(HERE, "libadasum.so")
# a measuring tool (the memory system's ceiling for the combine pass's access pattern)
CEILING_PATH = os.path.join(HERE, "pattern_ceiling")

# (source, defines): the resident kernels are compiled once per storage type of the gradients and range of worker counts
SOURCES = [("adasum_resident.hip", [f"-DADASUM_LEAF_TYPE={t}", f"-DADASUM_WIDE_GROUPS={w}"])
           for t, w in ((0, 0), (1, 0), (2, 0), (3, 0), (0, 1), (1, 1), (2, 1))] + [
    ("adasum_kernels.hip", []), ("adasum_api.cpp", []), ("adasum_plan.cpp", [])]

# -packed-fp32-ops off: the compiler must not form packed fp32 instructions.
DEVICE_FLAGS = ["--offload-arch=gfx950", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def hipcc() -> str:
    exe = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(exe):
        raise RuntimeError("hipcc not found; the HIP library cannot be built")
    return exe


def build_library(verbose: bool = True, extra_flags=(), out_path: str = LIB_PATH) -> str:
    """Compiles every source to an object (side by side: the resident kernels of the four storage types take most
    of the time) and links them."""
    flags = ["-O3", "-std=c++17", "-fPIC", "-fvisibility=hidden", "-Wall", "-Wno-unused-command-line-argument",
             *DEVICE_FLAGS, "-I", os.path.join(ROOT, "include"), "-I", CSRC, *extra_flags]
    with tempfile.TemporaryDirectory() as tmp:
        objects, commands = [], []
        for i, (source, defines) in enumerate(SOURCES):
            objects.append(os.path.join(tmp, f"{i}.o"))
            commands.append([hipcc(), *flags, *defines, "-c", os.path.join(CSRC, source), "-o", objects[-1]])

        def run(cmd):
            if verbose:
                print(" ".join(cmd), flush=True)
            subprocess.run(cmd, check=True)

        with ThreadPoolExecutor(min(len(commands), os.cpu_count() or 1, 8)) as pool:
            list(pool.map(run, commands))
        run([hipcc(), "-shared", "-fPIC", *DEVICE_FLAGS, "-Wno-unused-command-line-argument", *objects, "-o", out_path])
    return out_path


def build_pattern_ceiling(verbose: bool = True, out_path: str = CEILING_PATH) -> str:
    cmd = [hipcc(), "-O3", "-std=c++17", "-Wall", "-Wno-unused-command-line-argument", *DEVICE_FLAGS,
           os.path.join(CSRC, "pattern_ceiling.hip"), "-o", out_path]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    return out_path


if __name__ == "__main__":
    build_library()
    build_pattern_ceiling()
    print(LIB_PATH)
    print(CEILING_PATH)
    sys.exit(0)
