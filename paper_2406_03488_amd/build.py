"""Builds libs1f.so (HIP kernels + C ABI) in-tree with hipcc for gfx950."""
from __future__ import annotations

import os
import subprocess
import sysconfig

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(HERE, "csrc")
INCLUDE = os.path.join(os.path.dirname(HERE), "include")
LIB = os.path.join(HERE, "libs1f.so")
CALLS_LIB = os.path.join(HERE, "_torch_calls.so")   # the tensor calls of binding.py
PROBE_LIB = os.path.join(HERE, "libs1f_probe.so")   # measurement aid used by bench.py only

SOURCES = ["s1f_api.hip", "s1f_cache.hip", "s1f_partition.cpp", "s1f_schedule.cpp", "s1f_pipeline.cpp"]
FLAGS = ["--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared", "-Wall", "-Werror=array-bounds",
         # packed fp32 VALU forms are kept out of generated code on this target
         "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops"]


def build_library(verbose: bool = False) -> str:
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    cmd = [hipcc, *FLAGS, f"-I{INCLUDE}", f"-I{CSRC}", "-o", LIB, *[os.path.join(CSRC, s) for s in SOURCES]]
    proc = subprocess.run(cmd, capture_output=True, text=True)
    if proc.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + proc.stdout + proc.stderr)
    if verbose:
        print(proc.stderr)
    build_calls()
    cmd = [hipcc, *FLAGS, "-o", PROBE_LIB, os.path.join(CSRC, "mfma_peak.hip")]
    proc = subprocess.run(cmd, capture_output=True, text=True)
    if proc.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + proc.stdout + proc.stderr)
    return LIB


def build_calls() -> None:
    """The extension module of the tensor calls: host code against torch's headers."""
    import torch
    root = os.path.dirname(torch.__file__)
    include, lib = os.path.join(root, "include"), os.path.join(root, "lib")
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}", f"-I{INCLUDE}", f"-isystem{include}",
           f"-isystem{os.path.join(include, 'torch', 'csrc', 'api', 'include')}", f"-isystem{sysconfig.get_paths()['include']}",
           os.path.join(CSRC, "torch_calls.cpp"), "-o", CALLS_LIB, f"-L{lib}", "-ltorch_python", "-ltorch_cpu", "-lc10"]
    proc = subprocess.run(cmd, capture_output=True, text=True)
    if proc.returncode != 0:
        raise RuntimeError("g++ failed:\n" + proc.stdout + proc.stderr)


if __name__ == "__main__":
    print(build_library(verbose=True))
