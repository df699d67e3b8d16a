"""Build libmurmur.so for gfx950 (MI355X) from csrc/.

kernels.hip is compiled by hipcc for gfx950 only; api.cpp (host-only C ABI
layer) by g++.  The shared object lands next to this file, where the ctypes
binding loads it, and beside it the _pycall module, the argument converter of the
per-step calls (pycall.cpp), where Python's headers are there to build it; the
binding does without it.  Packed-fp32 instruction selection is disabled for
device code, and the first 16 kernel-argument dwords are preloaded into SGPRs.
Only the murmur_* entry points are exported.
"""
from __future__ import annotations

import glob
import os
import shutil
import subprocess
import sysconfig
import warnings

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
INCLUDE = os.path.join(ROOT, "include")
LIB = os.path.join(PKG, "libmurmur.so")
PYCALL = os.path.join(PKG, "_pycall" + sysconfig.get_config_var("EXT_SUFFIX"))  # for this interpreter only
BUILD_DIR = os.path.join(ROOT, "_build")
ARCH = "gfx950"


def _hipcc() -> str:
    for cand in (shutil.which("hipcc"), "/opt/rocm/bin/hipcc"):
        if cand and os.path.exists(cand):
            return cand
    raise RuntimeError("hipcc not found: the HIP toolchain (ROCm) is required to build libmurmur")


def _run(cmd: list[str]) -> None:
    res = subprocess.run(cmd, capture_output=True, text=True)
    if res.returncode != 0:
        raise RuntimeError(f"build step failed ({res.returncode}): {' '.join(cmd)}\n{res.stdout}\n{res.stderr}")


COMMON_FLAGS = ["-O3", "-std=c++17", "-fPIC", "-fvisibility=hidden", f"-I{INCLUDE}", f"-I{CSRC}", "-Wall"]
# Device code: packed-fp32 instruction selection off; the first 16 kernel-argument dwords preloaded into SGPRs.
KERNEL_FLAGS = [f"--offload-arch={ARCH}", *COMMON_FLAGS, "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
                "-mllvm", "-amdgpu-kernarg-preload-count=16"]


def _build_pycall(verbose: bool) -> None:
    """The argument converter.  None of an earlier build is left beside the new library, whose functions it would
    call by the old signatures."""
    for old in glob.glob(os.path.join(glob.escape(PKG), "_pycall*.so")):
        os.remove(old)
    tmp = PYCALL + ".tmp"
    cmd = ["g++", *COMMON_FLAGS, "-Wextra", "-shared", f"-I{sysconfig.get_paths()['include']}",
           os.path.join(CSRC, "pycall.cpp"), "-o", tmp]
    if verbose:
        print(" ".join(cmd), flush=True)
    try:
        _run(cmd)
    except RuntimeError as e:
        warnings.warn(f"the per-step calls will go through ctypes: {e}")
        return
    os.replace(tmp, PYCALL)


def build(verbose: bool = False) -> str:
    """Compile every source and link libmurmur.so (always rebuilds)."""
    os.makedirs(BUILD_DIR, exist_ok=True)
    hipcc = _hipcc()
    k_obj = os.path.join(BUILD_DIR, "kernels.o")
    a_obj = os.path.join(BUILD_DIR, "api.o")
    steps = [
        [hipcc, *KERNEL_FLAGS, "-c", os.path.join(CSRC, "kernels.hip"), "-o", k_obj],
        ["g++", *COMMON_FLAGS, "-Wextra", "-c", os.path.join(CSRC, "api.cpp"), "-o", a_obj],
    ]
    for cmd in steps:
        if verbose:
            print(" ".join(cmd), flush=True)
        _run(cmd)
    tmp = LIB + ".tmp"
    link = [hipcc, f"--offload-arch={ARCH}", "-shared", "-fPIC", k_obj, a_obj, "-o", tmp]
    if verbose:
        print(" ".join(link), flush=True)
    _run(link)
    os.replace(tmp, LIB)
    _build_pycall(verbose)
    return LIB


if __name__ == "__main__":
    print(build(verbose=True))
