"""Build libonmt.so (the gfx950 HIP kernels and the C ABI) in-tree with hipcc.

Usage: ``python -m paper_1805_11462_amd.build`` or ``paper_1805_11462_amd.build.build()``.
"""

import os
import shutil
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libonmt.so")
SOURCES = ["onmt_api.hip", "thin.hip", "gen.hip", "wide.hip", "attention.hip", "beam.hip"]

# Host code (weight packing) uses the fp16 conversion instructions that every host of such a card has.
# Packed-FP32 VALU ops are switched off for all device code (only plain fp32 VALU and MFMA are used).
HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Xarch_host", "-march=x86-64-v3", "-Wno-unused-result",
]


def hipcc_path():
    p = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(p):
        raise RuntimeError("hipcc not found; the HIP library cannot be built")
    return p


def build(verbose=False):
    srcs = [os.path.join(CSRC, s) for s in SOURCES]
    tmp = LIB + ".tmp"
    cmd = [hipcc_path(), *HIPCC_FLAGS, "-o", tmp, *srcs]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        sys.stderr.write(r.stdout + r.stderr)
        raise RuntimeError(f"hipcc failed with exit code {r.returncode}")
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
