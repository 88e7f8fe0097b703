"""Compile the HIP/C++ sources into the in-tree shared library libbires.so (gfx950)."""

import glob
import os
import subprocess
import tempfile
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libbires.so")

HIPCC_FLAGS = [
    "--offload-arch=gfx950",
    "-O3",
    "-fPIC",
    "-std=c++17",
    # no packed FP32 instructions anywhere in the device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
]

# Flags of single files.  ee.hip keeps its coefficient arrays in registers by
# compile-time indices; turning them into vector values first makes whole
# vectors move and spill (k_eval_elim_ee24: 176 bytes of scratch instead of none).
# kernels.hip is better with it: k_crt_mfma takes 100 registers, 120 without.
FILE_FLAGS = {"ee.hip": ["-mllvm", "-disable-promote-alloca-to-vector"]}


def sources():
    return sorted(glob.glob(os.path.join(CSRC, "*.hip")) + glob.glob(os.path.join(CSRC, "*.cpp")))


def build(verbose=False):
    """Always recompiles (the driver calls this as its build check)."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    tmp = LIB + ".tmp"

    def run(cmd):
        res = subprocess.run(cmd, capture_output=True, text=True)
        if res.returncode != 0:
            raise RuntimeError("hipcc failed:\n" + res.stdout + res.stderr)

    with tempfile.TemporaryDirectory() as objdir, ThreadPoolExecutor(min(8, os.cpu_count() or 1)) as pool:

        def compile_one(src):
            name = os.path.basename(src)
            obj = os.path.join(objdir, name + ".o")
            run([hipcc] + HIPCC_FLAGS + FILE_FLAGS.get(name, []) + ["-c", "-o", obj, src])
            return obj

        objs = list(pool.map(compile_one, sources()))
        run([hipcc, HIPCC_FLAGS[0], "-shared", "-fPIC", "-o", tmp] + objs)
    os.replace(tmp, LIB)
    if verbose:
        print("built", LIB)
    return LIB


if __name__ == "__main__":
    build(verbose=True)
