"""Build the native library ``liblbm_entropic.so`` with hipcc for gfx950.

Flags: -O3, C++17, FMA contraction off (the fused multiply-adds the kernels
want are written out, so every kernel variant rounds identically), packed-FP32
instructions disabled, code-object version 5.
"""
from __future__ import annotations

import glob
import os
import subprocess
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIB = os.path.join(HERE, "liblbm_entropic.so")

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared", "-ffp-contract=off",
         "-mcode-object-version=5", "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-Wall", "-Wno-unused-function"]


def sources():
    return sorted(glob.glob(os.path.join(HERE, "csrc", "*.hip")))


def build(verbose: bool = False) -> str:
    """Compile every source (side by side) and link them."""
    tmp = LIB + ".tmp"

    def hipcc(args):
        cmd = [HIPCC, *args]
        if verbose:
            print(" ".join(cmd), flush=True)
        r = subprocess.run(cmd, capture_output=True, text=True)
        noise = "is not a recognized feature for this target"
        err = "\n".join(l for l in r.stderr.splitlines() if noise not in l and l.strip() != "1 warning generated.")
        if r.returncode != 0:
            raise RuntimeError(f"hipcc failed ({r.returncode}):\n{err}")
        if verbose and err.strip():
            print(err)

    with tempfile.TemporaryDirectory() as d:
        objects = [os.path.join(d, os.path.basename(s) + ".o") for s in sources()]
        flags = [f for f in FLAGS if f != "-shared"] + ["-I" + os.path.join(ROOT, "include"),
                                                        "-I" + os.path.join(HERE, "csrc")]
        with ThreadPoolExecutor(len(objects)) as pool:
            list(pool.map(lambda so: hipcc([*flags, "-c", so[0], "-o", so[1]]), zip(sources(), objects)))
        hipcc(["--offload-arch=gfx950", "-shared", "-fPIC", *objects, "-o", tmp])
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
