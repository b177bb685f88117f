"""Builds ``libhyena.so`` (the C-ABI library of gfx950 kernels) in-tree with hipcc, and beside it, where torch's and Python's
headers and a C++ compiler are there, the native marshalling of the binding's calls (``_fastcall``, a CPython extension)."""
from __future__ import annotations

import hashlib
import os
import shutil
import subprocess
import sys
import sysconfig
import warnings
from concurrent.futures import ThreadPoolExecutor

PKG = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(PKG)
CSRC = os.path.join(PKG, "csrc")
OBJ_DIR = os.path.join(PKG, "_build")
LIB = os.path.join(PKG, "libhyena.so")

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


def _older(built: str, deps) -> bool:
    return not os.path.exists(built) or any(os.path.getmtime(d) > os.path.getmtime(built) for d in deps)


def _header() -> str:
    return os.path.join(ROOT, "include", "hyena.h")


def stale() -> bool:
    """True when the library is missing or older than any file it is built from."""
    return _older(LIB, [os.path.join(CSRC, f) for f in os.listdir(CSRC) if f != "fastcall.cpp"] + [_header()])


def fast_path() -> str:
    """The extension for the torch that is there.  It reads torch's objects by their layout, so its name says which torch
    (version, build, C++ ABI) it was built against, and no other finds it."""
    import torch

    key = "%s %s %d" % (torch.__version__, torch.version.git_version, torch.compiled_with_cxx11_abi())
    suffix = sysconfig.get_config_var("EXT_SUFFIX") or ".so"
    return os.path.join(PKG, "_fastcall_" + hashlib.sha1(key.encode()).hexdigest()[:10] + suffix)


def build_fastcall() -> str:
    """The extension's torch libraries are those that the importing torch has loaded (no run path)."""
    import torch
    from torch.utils.cpp_extension import include_paths, library_paths

    cxx = shutil.which(os.environ.get("CXX", "g++")) or os.path.join(os.path.dirname(_hipcc()), "..", "llvm", "bin", "clang++")
    path = fast_path()
    tmp = path + ".%d.tmp" % os.getpid()
    cmd = [cxx, "-O2", "-std=c++17", "-fPIC", "-shared", "-D_GLIBCXX_USE_CXX11_ABI=%d" % torch.compiled_with_cxx11_abi(),
           "-I" + os.path.join(ROOT, "include"), "-I" + sysconfig.get_paths()["include"]]
    cmd += ["-I" + d for d in include_paths()] + [os.path.join(CSRC, "fastcall.cpp"), "-o", tmp]
    cmd += ["-L" + d for d in library_paths()] + ["-ltorch_python", "-ltorch_cpu", "-lc10"]
    proc = subprocess.run(cmd, capture_output=True, text=True)
    if proc.returncode != 0:
        raise RuntimeError("%s failed on fastcall.cpp:\n%s" % (cxx, proc.stderr))
    os.replace(tmp, path)
    return path


_fast_failed = False


def ensure_fastcall(force: bool = False) -> str | None:
    """The extension's path, after building it where it is missing or out of date (or anyway).  Where it cannot be built the
    library does without it: a warning, once per process, and None."""
    global _fast_failed
    try:
        path = fast_path()
        if not force and not _older(path, [os.path.join(CSRC, "fastcall.cpp"), _header()]):
            return path
        return None if _fast_failed else build_fastcall()
    except Exception as e:  # no torch, headers or compiler, a directory that is not ours to write, an error in the source
        _fast_failed = True
        warnings.warn("native marshalling not built, calls are marshalled through ctypes: %s" % e, RuntimeWarning)
        return None


def build_library(verbose: bool = False) -> str:
    """Compile every kernel translation unit for gfx950 and link the shared library; build the extension beside it if it can
    be built."""
    os.makedirs(OBJ_DIR, exist_ok=True)
    with ThreadPoolExecutor(max_workers=min(8, len(SOURCES) + 1)) as pool:
        pool.submit(ensure_fastcall, True)
        objs = list(pool.map(_compile, SOURCES))
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
