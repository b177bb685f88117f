"""Builds ``libhyena.so`` (the C-ABI library of gfx950 kernels) in-tree with hipcc, and the native marshalling of the
binding's calls (``_fastcall``, a CPython extension against torch's headers)."""
from __future__ import annotations

import os
import shutil
import subprocess
import sys
import sysconfig
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
OBJ_DIR = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "libhyena.so")
FAST = os.path.join(PKG, "_fastcall" + (sysconfig.get_config_var("EXT_SUFFIX") or ".so"))

SOURCES = ["api.hip", "se_kernels.hip", "sew_kernels.hip", "direct_kernels.hip", "split_kernels.hip", "mr_kernels.hip", "cp_kernels.hip", "cp4_kernels.hip", "li_kernels.hip", "chain4_kernels.hip", "chain_bwd_kernels.hip", "bwd_kernels.hip", "bwdw_kernels.hip", "mr_bwd_kernels.hip", "cp4_bwd_kernels.hip", "yardstick_kernels.hip"]

# Packed-fp32 instruction selection is switched off for all device code in this library.
HIPCC_FLAGS = [
    "--offload-arch=gfx950", "-O3", "-std=c++17", "-fPIC",
    "-Xclang", "-target-feature", "-Xclang", "-packed-fp32-ops",
    "-I" + os.path.join(ROOT, "include"), "-I" + CSRC,
]


def _hipcc() -> str:
    return os.environ.get("HIPCC", "/opt/rocm/bin/hipcc" if os.path.exists("/opt/rocm/bin/hipcc") else "hipcc")


def _compile(src: str) -> str:
    obj = os.path.join(OBJ_DIR, src.replace(".hip", ".o"))
    cmd = [_hipcc()] + HIPCC_FLAGS + ["-c", os.path.join(CSRC, src), "-o", obj]
    proc = subprocess.run(cmd, capture_output=True, text=True)
    if proc.returncode != 0:
        raise RuntimeError("hipcc failed on %s:\n%s" % (src, proc.stderr))
    return obj


def stale() -> bool:
    """True when the library or the extension is missing or older than any file it is built from."""
    if not os.path.exists(LIB) or not os.path.exists(FAST):
        return True
    built = min(os.path.getmtime(LIB), os.path.getmtime(FAST))
    deps = [os.path.join(CSRC, f) for f in os.listdir(CSRC)] + [os.path.join(ROOT, "include", "hyena.h")]
    return any(os.path.getmtime(d) > built for d in deps)


def _build_fastcall() -> None:
    """The extension's torch libraries are those that the importing torch has loaded (no run path)."""
    import torch
    from torch.utils.cpp_extension import include_paths, library_paths

    cxx = shutil.which(os.environ.get("CXX", "g++")) or os.path.join(os.path.dirname(_hipcc()), "..", "llvm", "bin", "clang++")
    tmp = FAST + ".%d.tmp" % os.getpid()
    cmd = [cxx, "-O2", "-std=c++17", "-fPIC", "-shared", "-D_GLIBCXX_USE_CXX11_ABI=%d" % int(torch._C._GLIBCXX_USE_CXX11_ABI),
           "-I" + os.path.join(ROOT, "include"), "-I" + sysconfig.get_paths()["include"]]
    cmd += ["-I" + d for d in include_paths()] + [os.path.join(CSRC, "fastcall.cpp"), "-o", tmp]
    cmd += ["-L" + d for d in library_paths()] + ["-ltorch_python", "-ltorch_cpu", "-lc10"]
    proc = subprocess.run(cmd, capture_output=True, text=True)
    if proc.returncode != 0:
        raise RuntimeError("%s failed on fastcall.cpp:\n%s" % (cxx, proc.stderr))
    os.replace(tmp, FAST)


def build_library(verbose: bool = False) -> str:
    """Compile every kernel translation unit for gfx950 and link the shared library; build the extension beside it."""
    os.makedirs(OBJ_DIR, exist_ok=True)
    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES) + 1)) as pool:
        fast = pool.submit(_build_fastcall)
        objs = list(pool.map(_compile, SOURCES))
        fast.result()
    tmp = LIB + ".%d.tmp" % os.getpid()
    cmd = [_hipcc(), "--offload-arch=gfx950", "-shared", "-fPIC", "-o", tmp] + objs
    proc = subprocess.run(cmd, capture_output=True, text=True)
    if proc.returncode != 0:
        raise RuntimeError("link failed:\n%s" % proc.stderr)
    os.replace(tmp, LIB)
    if verbose:
        print("built", LIB, file=sys.stderr)
    return LIB


if __name__ == "__main__":
    build_library(verbose=True)
