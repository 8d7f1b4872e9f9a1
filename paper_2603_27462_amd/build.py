"""Builds librsr.so (HIP, gfx950 only) in-tree with hipcc, and the native part of the binding with g++."""
from __future__ import annotations

import os
import subprocess
import sys
import sysconfig
import warnings

PKG_DIR = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(PKG_DIR, "csrc")
INCLUDE = os.path.join(os.path.dirname(PKG_DIR), "include")
LIB_PATH = os.path.join(PKG_DIR, "librsr.so")
CALL_PATH = os.path.join(PKG_DIR, "_rsr_call.so")
SOURCES = ["rsr_api.hip", "rsr_preprocess.hip", "rsr_matvec.hip", "rsr_packed.hip", "rsr_probe.hip",
           "rsr_narrow.hip"]

HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC", "-shared",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    # the first kernel arguments (stream and vector pointers, geometry) arrive in registers
    # instead of through a scalar load at the start of every wave
    "-mllvm", "-amdgpu-kernarg-preload-count=14",
    "-Wall", "-Wno-unused-command-line-argument",
]


def _run(cmd, verbose: bool) -> None:
    if verbose:
        print(" ".join(cmd), file=sys.stderr)
    proc = subprocess.run(cmd, stdout=subprocess.PIPE, stderr=subprocess.STDOUT, text=True)
    if proc.returncode != 0:
        raise RuntimeError(cmd[0] + " failed:\n" + proc.stdout)
    if verbose and proc.stdout.strip():
        print(proc.stdout, file=sys.stderr)


def torch_tag() -> str:
    """The torch that the native part of the binding is compiled against; it uses that build's C++ classes."""
    import torch
    return "%s %s abi%d" % (torch.__version__, torch.version.git_version, int(torch._C._GLIBCXX_USE_CXX11_ABI))


def build_call(verbose: bool = False) -> str:
    """Compile the native part of the binding against the installed torch."""
    import torch
    root = os.path.dirname(torch.__file__)
    tmp = CALL_PATH + ".tmp%d" % os.getpid()
    cmd = [os.environ.get("CXX", "g++"), "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__=1",
           "-DUSE_ROCM=1", "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI),
           '-DRSR_TORCH="%s"' % torch_tag()]
    for path in (os.path.join(root, "include"), os.path.join(root, "include", "torch", "csrc", "api", "include"),
                 sysconfig.get_paths()["include"], os.path.join(os.environ.get("ROCM_PATH", "/opt/rocm"), "include")):
        cmd += ["-isystem", path]
    cmd += ["-I", INCLUDE, os.path.join(CSRC, "rsr_call.cpp"), "-L", os.path.join(root, "lib"), "-lc10", "-lc10_hip",
            "-ltorch_cpu", "-ltorch_python", "-o", tmp]
    _run(cmd, verbose)
    os.replace(tmp, CALL_PATH)
    return CALL_PATH


def build_library(verbose: bool = False) -> str:
    """Compile every HIP source into paper_2603_27462_amd/librsr.so, and the binding's native part if that can be
    compiled here: without it the binding calls the library through ctypes."""
    hipcc = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
    tmp = LIB_PATH + ".tmp%d" % os.getpid()
    cmd = [hipcc] + HIPCC_FLAGS + ["-I", INCLUDE, "-I", CSRC]
    cmd += [os.path.join(CSRC, s) for s in SOURCES] + ["-o", tmp]
    _run(cmd, verbose)
    os.replace(tmp, LIB_PATH)
    try:
        build_call(verbose)
    except (ImportError, OSError, RuntimeError) as e:
        if os.path.exists(CALL_PATH):
            os.remove(CALL_PATH)                # it would not be that of these sources
        warnings.warn("the native part of the binding is not built, small products will take longer: %s" % e)
    return LIB_PATH


def sources_newer_than_library() -> list:
    """Source files modified after the built library (empty when it is up to date or absent)."""
    if not os.path.exists(LIB_PATH):
        return []
    built = os.path.getmtime(LIB_PATH)
    files = [os.path.join(CSRC, f) for f in sorted(os.listdir(CSRC))]
    files.append(os.path.join(INCLUDE, "rsr.h"))
    return [os.path.relpath(f, os.path.dirname(PKG_DIR)) for f in files
            if f.endswith((".hip", ".h", ".cpp")) and os.path.getmtime(f) > built + 1.0]


if __name__ == "__main__":
    print(build_library(verbose=True))
