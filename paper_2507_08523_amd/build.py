"""Builds libilpc.so (host prefix cache + gfx950 kernels) in-tree with hipcc, and
the native part of the Python binding (_binding.so) against PyTorch's headers.

    python -m paper_2507_08523_amd.build

Every HIP translation unit is compiled for gfx950 only, with packed-fp32 VALU
instructions disabled (``-target-feature -packed-fp32-ops``; the host pass
warns that it does not know the feature, which is harmless).
"""
from __future__ import annotations

import os
import subprocess
import sys

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
LIB = os.path.join(PKG, "libilpc.so")
SOURCES = [os.path.join(PKG, "csrc", "prefix_cache.cpp"), os.path.join(PKG, "csrc", "pair_table.cpp"),
           os.path.join(PKG, "csrc", "schedule.cpp"),
           os.path.join(PKG, "csrc", "paged_attn.hip"), os.path.join(PKG, "csrc", "rope_append.hip"),
           os.path.join(PKG, "csrc", "decode_attn.hip"),
           os.path.join(PKG, "csrc", "attn_noalloc.hip")]
BINDING = os.path.join(PKG, "_binding.so")
BINDING_SOURCE = os.path.join(PKG, "csrc", "binding.cpp")
ARCH = "gfx950"


def hipcc() -> str:
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    return os.path.join(rocm, "bin", "hipcc")


def build_binding(verbose: bool = False) -> str:
    """Compile the native binding (host code only) against the torch that is installed (nothing
    without a HIP build of torch: no tensor is on a GPU then)."""
    import sysconfig

    try:
        import torch
    except ImportError:
        return ""
    if torch.version.hip is None:
        return ""

    t = os.path.dirname(torch.__file__)
    rocm = os.environ.get("ROCM_PATH", "/opt/rocm")
    tmp = BINDING + ".tmp"
    cmd = ["g++", "-O2", "-std=c++17", "-fPIC", "-shared", "-Wall", "-D__HIP_PLATFORM_AMD__", "-DUSE_ROCM",
           f"-D_GLIBCXX_USE_CXX11_ABI={int(torch._C._GLIBCXX_USE_CXX11_ABI)}",
           "-isystem", os.path.join(t, "include"),
           "-isystem", os.path.join(t, "include", "torch", "csrc", "api", "include"),
           "-isystem", os.path.join(rocm, "include"), "-isystem", sysconfig.get_paths()["include"],
           BINDING_SOURCE, "-L", os.path.join(t, "lib"), "-ltorch_python", "-ltorch", "-ltorch_cpu", "-lc10",
           "-lc10_hip", "-o", tmp]
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError("binding.cpp failed:\n" + res.stdout + res.stderr)
    if verbose and (res.stdout or res.stderr):
        print(res.stdout + res.stderr, file=sys.stderr)
    os.replace(tmp, BINDING)
    return BINDING


def build(verbose: bool = False) -> str:
    """Compile the library and the binding (always recompiles) and return the library's path.  Without
    a binding (no g++, no torch headers) the package still runs, its calls through ctypes."""
    tmp = LIB + ".tmp"
    cmd = [hipcc(), f"--offload-arch={ARCH}", "-O3", "-std=c++17", "-fPIC", "-shared",
           "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
           "-Wall", "-Wno-unused-result", "-Wno-inline-asm", "-I", os.path.join(ROOT, "include"),
           *SOURCES, "-o", tmp]
    res = subprocess.run(cmd, capture_output=True, text=True)
    noise = "is not a recognized feature for this target"
    msgs = [ln for ln in (res.stdout + res.stderr).splitlines() if noise not in ln]
    if res.returncode != 0:
        raise RuntimeError("hipcc failed:\n" + "\n".join(msgs))
    if verbose and msgs:
        print("\n".join(msgs), file=sys.stderr)
    os.replace(tmp, LIB)
    try:
        build_binding(verbose)
    except (OSError, RuntimeError) as e:
        if os.path.exists(BINDING):
            os.remove(BINDING)  # (of an earlier source)
        print(f"warning: no native binding: {e}", file=sys.stderr)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
