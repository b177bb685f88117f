"""Kernel sources run on the CPU (tests/host/emu: threads as fibers, the waves of a workgroup one after another between two
barriers), so that index arithmetic and missing barriers show without a GPU."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HOST = os.path.join(ROOT, "tests", "host")
CLANG = "/opt/rocm/llvm/bin/clang++"  # the kernels use its vector extensions


def run(name, line, tmp_path, *flags):
    if not os.path.exists(CLANG):
        pytest.skip("no clang++")
    exe = str(tmp_path / name)
    cmd = [CLANG, *flags, "-std=c++17", "-ffp-contract=off", "-x", "c++", "-I" + os.path.join(HOST, "emu"),
           "-I" + os.path.join(ROOT, "include"), "-I" + os.path.join(ROOT, "paper_2503_01868_amd", "csrc"),
           os.path.join(HOST, name + ".cpp"), "-o", exe]
    build = subprocess.run(cmd, capture_output=True, text=True)
    assert build.returncode == 0, build.stderr[-3000:]
    res = subprocess.run([exe], capture_output=True, text=True, timeout=600)
    assert res.returncode == 0 and line + ": 0 problem(s)" in res.stdout, (res.returncode, res.stdout[-5000:])


def test_fir_kernel_walks(tmp_path):
    """Walks over several tiles of the general FIR kernel give the bits of a plain loop, whichever wave runs ahead."""
    run("fir_emu", "fir emulation", tmp_path, "-O0")


def test_grouped_backward(tmp_path):
    """Gradients of batches and of rows beyond 24 bits, with nothing read or written outside the tensors."""
    run("mr_bwd_emu", "MR backward emulation", tmp_path, "-O1")


def test_split_products(tmp_path):
    """The general FIR on split bf16 products: fp32 precision at every magnitude, whichever wave runs ahead."""
    run("split_emu", "split emulation", tmp_path, "-O1")
