"""Build the HIP library of the batching path (librbatch.so) for gfx950.

Every source is compiled on each call (hipcc cross-compiles without a GPU);
objects go to a temporary directory, the shared library next to this file.
"""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "librbatch.so")
SOURCES = ["gemm.hip", "gemm_f32_split.hip", "kernels.hip", "runtime.cpp"]
ARCH = "gfx950"

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
CFLAGS = [
    "-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}",
    # packed fp32 instructions are kept out of the generated code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wno-unused-value", "-Wno-unused-result",
    f"-I{os.path.join(ROOT, 'include')}",
]


def build(verbose: bool = False) -> str:
    tmp = tempfile.mkdtemp(prefix="rbatch_build_")
    try:
        objs, jobs = [], []
        for src in SOURCES:  # all at once: the GEMM templates take minutes
            obj = os.path.join(tmp, src + ".o")
            cmd = [HIPCC, *CFLAGS, "-c", os.path.join(CSRC, src), "-o", obj]
            if verbose:
                print(" ".join(cmd), flush=True)
            jobs.append((cmd, subprocess.Popen(cmd, stderr=None if verbose else subprocess.DEVNULL)))
            objs.append(obj)
        for cmd, job in jobs:
            job.wait()
        for cmd, job in jobs:
            if job.returncode:
                raise subprocess.CalledProcessError(job.returncode, cmd)
        out_tmp = LIB + ".tmp"
        cmd = [HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", "-Wl,-z,defs", "-o", out_tmp, *objs, "-lpthread"]
        subprocess.run(cmd, check=True)
        os.replace(out_tmp, LIB)
    finally:
        shutil.rmtree(tmp, ignore_errors=True)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
