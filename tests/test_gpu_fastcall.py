"""The natively marshalled calls: the same bits as the binding's own path, and that path for whatever is not plain."""
import pytest
import torch
from torch.overrides import TorchFunctionMode

import paper_2503_01868_amd as hy
from paper_2503_01868_amd import binding

from gpu_util import say

pytestmark = pytest.mark.gpu


def acts(n, dtype, B=2, L=70, D=128):
    g = torch.Generator(device="cuda:0").manual_seed(n)
    return [torch.randn((B, L, D), generator=g, device="cuda:0").to(dtype) for _ in range(n)]


def table(rows, taps):
    return torch.randn((rows, taps), generator=torch.Generator(device="cuda:0").manual_seed(taps), device="cuda:0") * taps ** -0.5


def calls(dtype):
    dy, q, k, v = acts(4, dtype)
    lam = torch.rand((8, 5), generator=torch.Generator(device="cuda:0").manual_seed(3), device="cuda:0")
    f, h = table(128, 7), table(8, 40)
    return [("se_fwd", hy.hyena_se_fwd, (q, k, v, f, 1)), ("mr_fwd", hy.hyena_mr_fwd, (q, k, v, h)),
            ("se_bwd", hy.hyena_se_bwd, (dy, q, k, v, f)), ("mr_bwd", hy.hyena_mr_bwd, (dy, q, k, v, h, 16)),
            ("chain_fwd", hy.hyena_chain_fwd, (q, k, v, f, f, f, h)), ("li", hy.hyena_li_fwd, (q, k, v, table(8, 5), lam)),
            ("chain_bwd", hy.hyena_chain_bwd, (dy, q, k, v, f, f, f, h, 16, 1))]


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16], ids=["f32", "bf16"])
def test_the_same_bits(dtype, monkeypatch):
    binding.lib()
    assert binding._fast is not binding._Unmarshalled
    stream = torch.cuda.Stream()
    for name, fn, args in calls(dtype):
        say("marshalled %s %s" % (name, dtype))
        torch.cuda.synchronize()
        with torch.cuda.stream(stream):
            fast = fn(*args)
        stream.synchronize()
        with monkeypatch.context() as m:
            m.setattr(binding, "_fast", binding._Unmarshalled)
            slow = fn(*args)
        torch.cuda.synchronize()
        fast, slow = ((x,) if isinstance(x, torch.Tensor) else x for x in (fast, slow))
        assert isinstance(fast, tuple) and len(fast) == len(slow)
        for x, y in zip(fast, slow):
            assert torch.equal(x, y) and x.dtype == y.dtype and not x.requires_grad, name


class Seen(TorchFunctionMode):
    def __init__(self):
        self.names = []

    def __torch_function__(self, func, types, args=(), kwargs=None):
        self.names.append(getattr(func, "__name__", str(func)))
        return func(*args, **(kwargs or {}))


def test_what_is_not_plain_takes_the_other_path():
    q, k, v = acts(3, torch.float32)
    f = table(128, 7)
    binding.lib()
    for bad in ((q[:, ::2], k, v, f, 1), (q, k.half(), v, f, 1), (q, k, v[:1], f, 1), (q, k, v, f.double(), 1), (q, k, v, f, 3),
                (q.cpu(), k, v, f, 1), (q, k, v, f, 0), (None, k, v, f, 1)):
        assert binding._fast.gated(0, *bad) is None
        with pytest.raises(ValueError):
            hy.hyena_se_fwd(*bad)
    assert binding._fast.gated(0, q, k, v, f, True) is None  # (int(True) is a group of one all the same)
    with Seen() as seen:
        y = hy.hyena_se_fwd(q, k, v, f)
    assert "empty_like" in seen.names and torch.equal(y, hy.hyena_se_fwd(q, k, v, f))
    with pytest.raises(Exception):  # no storage behind a batched tensor, as before
        torch.func.vmap(lambda x: hy.hyena_se_fwd(x, x, x, f))(torch.stack([q, k]))
    with pytest.raises(binding.HyenaError):  # torch gives an empty tensor no address
        hy.hyena_se_fwd(q[:, :0], k[:, :0], v[:, :0], f)
    q.requires_grad_()
    assert not hy.hyena_se_fwd(q, k, v, f).requires_grad
