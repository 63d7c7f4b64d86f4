"""Build the gfx950 shared library libfe.so in-tree with hipcc."""
from __future__ import annotations

import concurrent.futures
import os
import subprocess
import sys
import tempfile

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
OUT = os.path.join(HERE, "libfe.so")
SOURCES = ["fe_api.cpp", "fe_refelem.cpp", "fe_dense.cpp", "fe_adjoint.cpp", "fe_tensor_rules.cpp", "fe_kernels.hip",
           "fe_nonlocal.hip", "fe_density.hip", "fe_lanczos.hip", "fe_poisson.hip"]
# the tensor-product kernels, one object per degree: by far the longest to compile
DEGREES = range(1, 8)
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-ffp-contract=off", "-Wall", "-Wno-unused-result",
]
LIBS = ["-L/opt/rocm/lib", "-lrocblas", "-lrocsolver", "-Wl,-rpath,/opt/rocm/lib"]
JOBS = int(os.environ.get("MAX_JOBS") or 0) or min(8, os.cpu_count() or 1)


def build(verbose: bool = False) -> str:
    """Compile every source (several at a time) and link libfe.so."""
    with tempfile.TemporaryDirectory(prefix="fe_build_") as tmpdir:
        jobs = [("fe_tensor.hip", f"fe_tensor_p{p}.o", [f"-DFE_TENSOR_DEGREE={p}"]) for p in reversed(DEGREES)]
        jobs += [(s, s + ".o", []) for s in SOURCES]

        def compile_one(job):
            src, obj, extra = job
            cmd = [HIPCC] + FLAGS + extra + ["-c", os.path.join(CSRC, src), "-o", os.path.join(tmpdir, obj)]
            if verbose:
                print(" ".join(cmd), flush=True)
            subprocess.check_call(cmd)
            return cmd[-1]

        with concurrent.futures.ThreadPoolExecutor(JOBS) as pool:
            objs = list(pool.map(compile_one, jobs))
        tmp = OUT + ".tmp"
        subprocess.check_call([HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs + LIBS)
        os.replace(tmp, OUT)
    return OUT


if __name__ == "__main__":
    build(verbose="-v" in sys.argv)
    print(OUT)
