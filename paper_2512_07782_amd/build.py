"""Build libgfwa.so (HIP kernels + C ABI) and the native Python binding in-tree for gfx950 with hipcc."""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
LIB = os.path.join(HERE, "libgfwa.so")
CALL_LIB = os.path.join(HERE, "_gfwa_call.so")  # the native half of the Python binding (host code only)
SOURCES = ["api.hip", "gate_scan.hip", "fp32_path.hip", "fwd_bf16.hip", "fwd_split_bf16.hip", "key_reach.hip", "bwd_bf16.hip", "bwd_split_bf16.hip", "decode.hip", "probe.hip"]
FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-fno-gpu-rdc",
    # packed fp32 VALU ops are kept off on the test machines
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-Wall", "-Wno-unused-function",
]


# per-file additions
EXTRA_FLAGS = {
    # MFMA results that the vector unit reads next (S, dP) stay in ordinary VGPRs instead of taking a
    # round trip through the accumulator registers
    "bwd_bf16.hip": ["-mllvm", "-amdgpu-mfma-vgpr-form"],
}


def build(verbose: bool = False, jobs: int = 10) -> str:
    """Compile every source to an object (in parallel), link the shared library, and build the native binding."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    objdir = os.path.join(HERE, "_build")
    os.makedirs(objdir, exist_ok=True)
    procs = [("binding.cpp", _spawn(_binding_cmd(), verbose))]
    objs = []
    for src in SOURCES:
        obj = os.path.join(objdir, src.replace(".hip", ".o"))
        objs.append(obj)
        cmd = [hipcc] + FLAGS + EXTRA_FLAGS.get(src, []) + ["-c", os.path.join(CSRC, src), "-o", obj]
        procs.append((src, _spawn(cmd, verbose)))
        if len(procs) >= jobs:
            _drain(procs, verbose)
    _drain(procs, verbose)
    cmd = [hipcc, "--offload-arch=gfx950", "-shared", "-fPIC", "-o", LIB] + objs
    subprocess.run(cmd, check=True)
    return LIB


def build_binding(verbose: bool = False) -> str:
    """Compile the native half of the Python binding alone (build() does it too)."""
    _drain([("binding.cpp", _spawn(_binding_cmd(), verbose))], verbose)
    return CALL_LIB


def _binding_cmd():
    import torch
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    root = os.path.dirname(torch.__file__)
    lib = os.path.join(root, "lib")
    return [os.environ.get("CXX", "g++"), os.path.join(CSRC, "binding.cpp"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
            "-D__HIP_PLATFORM_AMD__=1", "-DUSE_ROCM=1", "-isystem", os.path.join(rocm, "include"), "-isystem", os.path.join(root, "include"),
            "-isystem", os.path.join(root, "include", "torch", "csrc", "api", "include"),
            "-I" + sysconfig.get_paths()["include"], "-o", CALL_LIB, "-L" + lib, "-Wl,-rpath," + lib,
            "-lc10", "-lc10_hip", "-ltorch_cpu", "-ltorch_hip", "-ltorch_python"]


def _spawn(cmd, verbose):
    if verbose:
        print(" ".join(cmd), flush=True)
    return subprocess.Popen(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)


def _drain(procs, verbose):
    while procs:
        src, p = procs.pop(0)
        out, _ = p.communicate()
        out = "\n".join(l for l in out.splitlines() if "not a recognized feature" not in l)
        if p.returncode != 0:
            raise RuntimeError(f"compiling {src} failed:\n{out}")
        if out.strip() and (verbose or "warning:" in out):  # warnings are always shown
            print(out, flush=True)


if __name__ == "__main__":
    print(build(verbose="-v" in sys.argv))
