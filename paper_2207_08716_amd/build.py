"""Build the HIP library (libptporo.so) in-tree for gfx950 with hipcc."""
from __future__ import annotations

import os
import subprocess
import tempfile
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
LIB = os.path.join(PKG, "libptporo.so")
# One compiler run each; iter_kernel.hip in three parts (its many sweep kernels).
SOURCES = ["api.hip", "iter_kernel.hip", "refresh_kernel.hip", "aux_kernels.hip", "adjoint_kernels.hip", "waves.hip",
           "mg_kernels.hip", "krylov_kernels.hip"]

FLAGS = [
    "-O3", "-std=c++17", "-fPIC", "--offload-arch=gfx950",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


def build(verbose: bool = False, extra=None) -> str:
    """Compile every source into libptporo.so (always recompiles)."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    tmp = LIB + ".tmp"
    inc = ["-I", os.path.join(ROOT, "include"), "-I", CSRC]
    with tempfile.TemporaryDirectory() as objs:
        # one compiler per source, side by side
        def compile_one(job):
            src, part = job
            obj = os.path.join(objs, f"{src}.{part}.o")
            define = [] if part is None else [f"-DSWEEP_PART={part}"]
            cmd = [hipcc, *FLAGS, *(extra or []), *define, *inc, "-c", os.path.join(CSRC, src), "-o", obj]
            if verbose:
                print(" ".join(cmd))
            subprocess.run(cmd, check=True)
            return obj

        jobs = [(s, p) for s in SOURCES for p in (range(3) if s == "iter_kernel.hip" else (None,))]
        with ThreadPoolExecutor(max_workers=min(len(jobs), os.cpu_count() or 1)) as pool:
            built = list(pool.map(compile_one, jobs))
        link = [hipcc, "-shared", "--offload-arch=gfx950", *built, "-o", tmp]
        if verbose:
            print(" ".join(link))
        subprocess.run(link, check=True)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
