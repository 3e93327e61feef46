"""Build the gfx950 shared library (the C ABI declared in include/rt.h).

    python paper_2303_11103_amd/build.py

compiles every HIP and C++ source under ``csrc/`` with hipcc for gfx950 into
``paper_2303_11103_amd/librt_mi355x.so``.  Packed fp32 instructions are
disabled and float atomics use the hardware instructions.
"""
from __future__ import annotations

import glob
import os
import subprocess
import sys
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIB = os.path.join(HERE, "librt_mi355x.so")
ARCH = os.environ.get("RT_OFFLOAD_ARCH", "gfx950")


def sources():
    return sorted(glob.glob(os.path.join(HERE, "csrc", "*.hip"))) + sorted(glob.glob(os.path.join(HERE, "csrc", "*.cpp")))


# Flags of single files.  The fp64 antenna functions of the gradients hold some
# hundred polynomial coefficients; hoisted out of the kernels' loops into
# registers they leave one wave per SIMD (276 registers) instead of three.
FILE_FLAGS = {"grad.hip": ["-mllvm", "-disable-machine-licm"]}


def build(verbose: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    flags = ["--offload-arch=" + ARCH, "-O3", "-std=c++17", "-fPIC", "-munsafe-fp-atomics",
             "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops", "-I", os.path.join(ROOT, "include")]
    tmp = LIB + ".tmp%d" % os.getpid()
    with tempfile.TemporaryDirectory() as objs:
        def run(cmd):
            if verbose:
                print(" ".join(cmd), flush=True)
            subprocess.check_call(cmd)

        def compile_one(src):
            name = os.path.basename(src)
            obj = os.path.join(objs, name + ".o")
            run([hipcc, *flags, *FILE_FLAGS.get(name, []), "-c", src, "-o", obj])
            return obj

        with ThreadPoolExecutor(min(8, os.cpu_count() or 1)) as pool:
            made = list(pool.map(compile_one, sources()))
        run([hipcc, "--offload-arch=" + ARCH, "-shared", "-fPIC", *made, "-o", tmp])
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
