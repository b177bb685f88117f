"""The binding takes the current GPU and stream as plain numbers from torch's own bindings, which are not part of its
public interface, and does without them where a torch has other names for them."""
import importlib.util
import types

import pytest
import torch

from paper_2503_01868_amd import binding


@pytest.mark.parametrize("missing", [(), ("_cuda_getCurrentRawStream",), ("_cuda_getDevice",),
                                     ("_cuda_getCurrentRawStream", "_cuda_getDevice")], ids=lambda m: "+".join(m) or "none")
def test_current_gpu_and_stream(monkeypatch, missing):
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda device: 1000 + device, raising=False)
    monkeypatch.setattr(torch._C, "_cuda_getDevice", lambda: 1, raising=False)
    for name in missing:
        monkeypatch.delattr(torch._C, name)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda device=None: types.SimpleNamespace(cuda_stream=1000 + device))
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 1)
    spec = importlib.util.spec_from_file_location("binding_again", binding.__file__)
    again = importlib.util.module_from_spec(spec)
    again.__package__ = binding.__package__
    spec.loader.exec_module(again)

    def on_gpu(i):
        return types.SimpleNamespace(is_cuda=True, get_device=lambda: i, device=torch.device("cuda", i))

    assert again._stream(on_gpu(3), None) == 1003
    assert again._stream(on_gpu(3), 7) == 7 and again._stream(on_gpu(3), types.SimpleNamespace(cuda_stream=8)) == 8
    assert again._on(on_gpu(1)) is again._HERE
    assert isinstance(again._on(on_gpu(0)), torch.cuda.device)
