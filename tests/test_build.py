"""The native marshalling is an extra: the library builds and loads without it, and another torch does not find it."""
import importlib.util
import os
import subprocess

import pytest
import torch

from paper_2503_01868_amd import binding, build


@pytest.fixture
def no_extension(monkeypatch, tmp_path):
    """Nothing built for this torch, and no compiler that can (the binding's own is loaded before)."""
    binding.lib()
    monkeypatch.setattr(build, "fast_path", lambda: str(tmp_path / "_fastcall.so"))
    monkeypatch.setattr(build, "_fast_failed", False)
    monkeypatch.setenv("CXX", "false")


def test_library_loads_without_the_extension(no_extension):
    assert not build.stale()
    spec = importlib.util.spec_from_file_location("binding_without", binding.__file__)
    again = importlib.util.module_from_spec(spec)
    again.__package__ = binding.__package__
    spec.loader.exec_module(again)
    with pytest.warns(RuntimeWarning, match="marshalled through ctypes"):
        assert again.version() == binding.version()
    assert again._fast is again._Unmarshalled and again._fast.gated(0, None, None, None, None, 1) is None


def test_library_builds_without_the_extension(no_extension, monkeypatch, tmp_path):
    lib = str(tmp_path / "libhyena.so")
    ran = []

    def run(cmd, **kwargs):
        ran.append(cmd[0])
        if "-o" in cmd and "fastcall" not in " ".join(cmd):
            open(cmd[cmd.index("-o") + 1], "w").close()
        return subprocess.CompletedProcess(cmd, 1 if "fastcall" in " ".join(cmd) else 0, "", "no such header")

    monkeypatch.setattr(build, "LIB", lib)
    monkeypatch.setattr(build, "_compile", lambda src: src)
    monkeypatch.setattr(build.subprocess, "run", run)
    with pytest.warns(RuntimeWarning, match="no such header"):
        assert build.build_library() == lib
    assert os.path.exists(lib) and len(ran) == 2


def test_another_torch_has_another_extension(monkeypatch):
    paths = {build.fast_path()}
    for where, name, other in ((torch, "__version__", "2.10.1"), (torch.version, "git_version", "0" * 40),
                               (torch, "compiled_with_cxx11_abi", lambda: not torch._C._GLIBCXX_USE_CXX11_ABI)):
        with monkeypatch.context() as m:
            m.setattr(where, name, other)
            paths.add(build.fast_path())
    assert len(paths) == 4
