"""Builds the HIP library for gfx950 in-tree: paper_1811_12019_amd/libkfac_hip.so."""
from __future__ import annotations

import os
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

PKG_DIR = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(PKG_DIR, "csrc")
LIB_PATH = os.path.join(PKG_DIR, "libkfac_hip.so")
SOURCES = ["factor_bf16.hip", "factor_f16.hip", "factor_f32.hip", "factor.hip", "factor_finish.hip", "ema.hip", "packed.hip", "diff.hip", "update.hip", "bn.hip", "inverse.hip", "damping.hip", "precondition.hip", "runtime.hip"]
HIPCC_FLAGS = [
    "-O3", "--offload-arch=gfx950", "-fPIC", "-std=c++17",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",   # no packed-fp32 VALU ops
    "-Wall", "-Wno-unused-function",
]


def build(verbose: bool = False) -> str:
    """Compile every kernel source into one shared library; returns its path.  Raises on failure."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    extra = os.environ.get("KFAC_EXTRA_HIPCC_FLAGS", "").split()

    def run(cmd):
        proc = subprocess.run(cmd, capture_output=True, text=True)
        # the host pass does not know the gfx-only target feature and says so; that line is noise
        err = "\n".join(l for l in proc.stderr.splitlines() if "packed-fp32-ops" not in l)
        if proc.returncode != 0:
            raise RuntimeError("hipcc failed:\n" + " ".join(cmd) + "\n" + err)
        if verbose and err.strip():
            print(err, file=sys.stderr)

    with tempfile.TemporaryDirectory(prefix="kfac_build_") as tmp:
        objs = [os.path.join(tmp, s + ".o") for s in SOURCES]
        with ThreadPoolExecutor(min(8, os.cpu_count() or 1)) as pool:
            list(pool.map(lambda so: run([hipcc] + HIPCC_FLAGS + extra + ["-c", os.path.join(CSRC, so[0]), "-o", so[1]]), zip(SOURCES, objs)))
        run([hipcc, "--offload-arch=gfx950", "-shared", "-o", LIB_PATH] + objs)
    return LIB_PATH


if __name__ == "__main__":
    print(build(verbose=True))
