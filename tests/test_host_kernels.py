"""Kernel sources run on the CPU (tests/host/emu: threads as fibers, the waves of a workgroup one after another between two
barriers), so that index arithmetic and missing barriers show without a GPU."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HOST = os.path.join(ROOT, "tests", "host")
CLANG = "/opt/rocm/llvm/bin/clang++"  # the kernels use its vector extensions


def test_fir_kernel_walks(tmp_path):
    """Walks over several tiles of the general FIR kernel give the bits of a plain loop, whichever wave runs ahead."""
    if not os.path.exists(CLANG):
        pytest.skip("no clang++")
    exe = str(tmp_path / "fir_emu")
    cmd = [CLANG, "-O0", "-std=c++17", "-ffp-contract=off", "-x", "c++", "-I" + os.path.join(HOST, "emu"),
           "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(ROOT, "paper_2503_01868_amd", "csrc"),
           os.path.join(HOST, "fir_emu.cpp"), "-o", exe]
    build = subprocess.run(cmd, capture_output=True, text=True)
    assert build.returncode == 0, build.stderr[-3000:]
    res = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    assert res.returncode == 0 and "fir emulation: 0 problem(s)" in res.stdout, res.stdout[-5000:]
