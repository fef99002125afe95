"""Build the HIP library liblb.so (gfx950) in-tree.

Each translation unit compiles in its own hipcc process (the four population
formats instantiate their kernels separately), then one shared library is
linked.  Packed-FP32 code generation is disabled for all device code.
"""
import os
import subprocess
import sys
from concurrent.futures import ThreadPoolExecutor

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
CSRC = os.path.join(HERE, "csrc")
BUILD = os.path.join(HERE, "_build")
LIB = os.path.join(HERE, "liblb.so")
SOURCES = ["lb_api.hip", "common.hip", "kern_f64.hip", "kern_f64_pow.hip", "kern_f32.hip", "kern_f16.hip",
           "kern_bf16.hip", "lb3_api.hip", "kern3_f64.hip", "kern3_f32.hip",
           "kern3_f16.hip", "kern3_bf16.hip", "sweep3x2.hip"]
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ARCH = "gfx950"
# No floating-point contraction: a node's arithmetic then compiles to the same
# roundings in every kernel that runs it (single-step and multi-step sweeps give
# bit-identical states); operations meant to be fused are written as fma calls.
FLAGS = ["-O3", "-std=c++17", "-fPIC", f"--offload-arch={ARCH}", "-Wall", "-Wno-unused-function",
         "-ffp-contract=off",
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
         "-I", os.path.join(ROOT, "include"), "-I", CSRC]
# The 16-bit sweeps are bound by vector issue; the instruction scheduler's
# ILP strategy gave a batch of 201 FP16 domains (185 M sites), two steps a
# launch, 0.967 against 0.981 ms per step (FP32 kernels keep the default:
# 1.593 against 1.584 ms with it).
# Without machine-level hoisting out of loops the FP64 kernels with pow keep to
# their registers (power law n = 1.3 in sheared flow, us a step: 1031 x 1000
# 44 -> 27, 2048^2 215 -> 103); the other FP64 kernels are up to 5 % slower so.
FILE_FLAGS = {"kern_f64_pow.hip": ["-mllvm", "-disable-machine-licm"],
              "kern_f16.hip": ["-mllvm", "-amdgpu-sched-strategy=max-ilp"],
              "kern_bf16.hip": ["-mllvm", "-amdgpu-sched-strategy=max-ilp"]}


def _compile(src: str, verbose: bool) -> str:
    obj = os.path.join(BUILD, os.path.splitext(src)[0] + ".o")
    cmd = [HIPCC, *FLAGS, *FILE_FLAGS.get(src, []), "-c", os.path.join(CSRC, src), "-o", obj]
    if verbose:
        print(" ".join(cmd), flush=True)
    r = subprocess.run(cmd, capture_output=True, text=True)
    if r.returncode != 0:
        raise RuntimeError(f"hipcc failed on {src}:\n{r.stdout}\n{r.stderr}")
    errs = [ln for ln in r.stderr.splitlines()
            if "warning" in ln and "packed-fp32-ops" not in ln and "feature" not in ln]
    if verbose and errs:
        print("\n".join(errs))
    return obj


def build(verbose: bool = False, jobs: int = 8) -> str:
    os.makedirs(BUILD, exist_ok=True)
    with ThreadPoolExecutor(max_workers=jobs) as ex:
        objs = list(ex.map(lambda s: _compile(s, verbose), SOURCES))
    tmp = LIB + ".tmp"
    cmd = [HIPCC, f"--offload-arch={ARCH}", "-shared", "-fPIC", *objs, "-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(tmp, LIB)
    return LIB


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
