"""Build the HIP shared library (gfx950) that implements the C ABI of include/lb.h.

Run as ``python -m paper_1402_6019_amd.build``; the result is ``liblb355.so`` next to this
file (in-tree, so it travels with the source tree).
"""

import os
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "liblb355.so")
SOURCES = ["lb_step_bf16.hip", "lb_step_f64.hip", "lb_step_f32.hip", "lb_tile_f64.hip", "lb_tile_f32.hip", "lb_tile_bf16.hip", "lb_tile_bf16sr.hip",
           "lb_kernels.hip", "lb_adjoint.hip", "lb_static.hip", "lb3_kernels.hip", "lb3_march.hip", "lb3_split.hip", "lb_api.cpp", "lb_batch.cpp", "lb_rheology.cpp", "lb3_api.cpp"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

FLAGS = [
    "--offload-arch=gfx950",
    "-O3",
    "-std=c++17",
    "-fPIC",
    "-shared",
    # packed FP32 instructions are kept out of all device code
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # no implicit contraction: the kernels write their fused multiply-adds explicitly, so
    # every kernel and launch shape rounds identically
    "-ffp-contract=off",
    "-Wall",
    "-Wno-unused-result",
    "-I" + os.path.join(ROOT, "include"),
]


def build(verbose=False):
    """Compile every source to an object file in parallel (one hipcc per source), then link."""
    from concurrent.futures import ThreadPoolExecutor
    objdir = os.path.join(ROOT, "_build")
    os.makedirs(objdir, exist_ok=True)
    compile_flags = [f for f in FLAGS if f != "-shared"]

    def compile_one(src):
        obj = os.path.join(objdir, os.path.splitext(src)[0] + ".o")
        cmd = [HIPCC, *compile_flags, "-c", os.path.join(CSRC, src), "-o", obj]
        if verbose:
            print(" ".join(cmd), flush=True)
        subprocess.run(cmd, check=True)
        return obj

    with ThreadPoolExecutor(max_workers=min(len(SOURCES), os.cpu_count() or 1)) as ex:
        objs = list(ex.map(compile_one, SOURCES))
    tmp = LIB + ".tmp"
    cmd = [HIPCC, "--offload-arch=gfx950", "-shared", "-fPIC", *objs, "-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    build(verbose="-v" in sys.argv)
    print(LIB)
