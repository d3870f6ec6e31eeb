"""Build libqgbe.so (HIP for gfx950) in-tree with hipcc."""
from __future__ import annotations

import glob
import os
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
LIB = os.path.join(PKG, "libqgbe.so")

HIPCC_FLAGS = [
    "-O3", "-std=c++17", "-fPIC", "--offload-arch=gfx950",
    # packed FP32 instructions stay off (hipcc forms them from scalar code otherwise)
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]


def sources() -> list[str]:
    csrc = os.path.join(PKG, "csrc")
    return sorted(glob.glob(os.path.join(csrc, "*.hip")) + glob.glob(os.path.join(csrc, "*.cpp")))


def build(verbose: bool = False) -> str:
    """Compile every HIP source of the library (always recompiles; the sources
    side by side) and link them."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    tmp = LIB + ".tmp"
    noise = "is not a recognized feature for this target"

    def hip(args):
        res = subprocess.run([hipcc, *args], capture_output=True, text=True)
        msgs = [l for l in (res.stdout + res.stderr).splitlines() if noise not in l]
        if res.returncode != 0:
            raise RuntimeError("hipcc failed:\n" + "\n".join(msgs))
        return msgs

    with tempfile.TemporaryDirectory() as objs, ThreadPoolExecutor(os.cpu_count() or 1) as pool:
        inc = ["-I", os.path.join(ROOT, "include"), "-I", os.path.join(PKG, "csrc")]
        srcs = sources()
        outs = [os.path.join(objs, os.path.basename(s) + ".o") for s in srcs]
        msgs = sum(pool.map(lambda so: hip([*HIPCC_FLAGS, *inc, "-c", so[0], "-o", so[1]]), zip(srcs, outs)), [])
        msgs += hip(["-shared", "-fPIC", "--offload-arch=gfx950", "-o", tmp, *outs])
    if verbose and msgs:
        print("\n".join(msgs), file=sys.stderr)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
