"""Compile librv.so (the gfx950 HIP library) and librv_synth.so (the seeded stream
generator used by the benchmark) in-tree with hipcc, and _rv_bind.so (the argument
marshalling of rv.py, a CPython module over torch's headers) with the host compiler."""
import os
import subprocess
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "librv.so")
SYNTH_LIB = os.path.join(HERE, "librv_synth.so")
BIND_LIB = os.path.join(HERE, "_rv_bind.so")
ARCH = os.environ.get("RV_OFFLOAD_ARCH", "gfx950")

HIPCC_FLAGS = [
    "-O3", "-std=c++17", "-fPIC", "-shared", f"--offload-arch={ARCH}",
    # keep the compiler from forming packed fp32 (v_pk_*_f32) instructions
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-result",
]
# The kernels take finite inputs: no NaN-quieting canonicalisation around min/max.
KERNEL_FLAGS = ["-fno-honor-nans", "-Xarch_device", "-mno-amdgpu-ieee"]


def _hipcc(out, sources, verbose, extra=()):
    cmd = ["hipcc", *HIPCC_FLAGS, *extra, "-o", out + ".tmp", *sources]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(out + ".tmp", out)


def _build_bind(verbose):
    import torch
    root = os.path.dirname(os.path.abspath(torch.__file__))
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           "-I" + sysconfig.get_paths()["include"], "-isystem", os.path.join(root, "include"), "-isystem",
           os.path.join(root, "include", "torch", "csrc", "api", "include"), os.path.join(CSRC, "rv_bind.cpp"),
           "-L" + os.path.join(root, "lib"), "-ltorch_python", "-ltorch_cpu", "-lc10",
           "-o", BIND_LIB + ".tmp"]
    if verbose:
        print(" ".join(cmd), flush=True)
    subprocess.run(cmd, check=True)
    os.replace(BIND_LIB + ".tmp", BIND_LIB)


def build(verbose: bool = False):
    _hipcc(LIB, [os.path.join(CSRC, f) for f in ("rv_host.cpp", "rv_plan.cpp", "attend.hip", "admit.hip")], verbose,
           KERNEL_FLAGS)
    _hipcc(SYNTH_LIB, [os.path.join(CSRC, "synth_gpu.hip")], verbose)
    _build_bind(verbose)
    return LIB, SYNTH_LIB


if __name__ == "__main__":
    print(build(verbose=True))
