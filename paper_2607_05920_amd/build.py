"""Build the HIP library libfhe_mi355x.so in place (gfx950 only)."""
from __future__ import annotations

import os
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIB = os.path.join(HERE, "libfhe_mi355x.so")
SOURCES = ["api.hip", "kernels.hip", "ntt_whole.hip", "lift_cols.hip", "rows_mid.hip", "crt_cols.hip", "ops.hip", "encode.cpp", "boot.cpp"]


def hipcc() -> str:
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    return os.path.join(rocm, "bin", "hipcc")


def build(verbose: bool = False) -> str:
    """Compile every source (side by side) and link the shared library; returns its path."""
    flags = [
        "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
        # packed FP32 instructions are kept out of every code object
        "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
        # the reconstruction and lift kernels unroll their k-block and tile loops fully
        "-mllvm", "-pragma-unroll-threshold=1000000",
        "-Wno-unused-result", "-Wno-unused-value", "-Wno-unused-command-line-argument",
        "-I", os.path.join(ROOT, "include"), "-I", os.path.join(HERE, "csrc"),
    ]

    def run(cmd):
        return subprocess.run(cmd, capture_output=True, text=True)

    with tempfile.TemporaryDirectory() as tmp:
        objs = [os.path.join(tmp, s + ".o") for s in SOURCES]
        # -cuid: the same code objects for the same sources, whatever the temporary folder is called
        jobs = [[hipcc(), *flags, "-cuid=" + s.split(".")[0], "-c", "-o", o, os.path.join(HERE, "csrc", s)]
                for s, o in zip(SOURCES, objs)]
        with ThreadPoolExecutor(min(len(jobs), os.cpu_count() or 1)) as pool:
            res = list(pool.map(run, jobs))
        if all(r.returncode == 0 for r in res):
            res.append(run([hipcc(), "--offload-arch=gfx950", "-shared", "-o", LIB + ".tmp", *objs]))
    err = "".join(r.stdout + r.stderr for r in res)
    if any(r.returncode != 0 for r in res):
        sys.stderr.write(err)
        raise RuntimeError("hipcc failed")
    if verbose:
        sys.stderr.write(err)
    os.replace(LIB + ".tmp", LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
