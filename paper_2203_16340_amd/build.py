"""Builds liblbfgsb.so (the HIP kernels and their C-ABI) in-tree for gfx950."""
from __future__ import annotations

import os
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "liblbfgsb.so")
SOURCES = ["fused.hip", "narrow.hip", "small.hip", "symmetric.hip", "gram.hip", "api.hip", "apass.hip", "resident.hip", "transport.hip", "vec.hip"]
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fno-gpu-rdc",
    # packed-fp32 instructions are kept out of the generated code on purpose
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-command-line-argument", "-Wno-unknown-warning-option",
]


def build(verbose: bool = False, extra_flags=()) -> str:
    """One object per source, up to four at a time, then the shared library."""
    with tempfile.TemporaryDirectory() as tmp:
        def compile_one(name: str) -> str:
            obj = os.path.join(tmp, name + ".o")
            cmd = ["hipcc", *FLAGS, *extra_flags, "-I", os.path.join(HERE, "..", "include"), "-c",
                   os.path.join(CSRC, name), "-o", obj]
            if verbose:
                print(" ".join(cmd), flush=True)
            subprocess.run(cmd, check=True)
            return obj

        with ThreadPoolExecutor(4) as pool:
            objects = list(pool.map(compile_one, SOURCES))
        subprocess.run(["hipcc", "--offload-arch=gfx950", "-shared", "-fPIC", *objects, "-o", LIB], check=True)
    return LIB


if __name__ == "__main__":
    build(verbose=True, extra_flags=sys.argv[1:])
