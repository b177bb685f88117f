"""The general FIR on split bf16 products (fp32 precision; filters shared by 8 or 16 adjacent channels) at the edges of its
chunks of 64 steps, its blocks of 64 channels and its windows of 2 to 5 source blocks; what is not finite, and what only
rounds to infinity as a bf16 head, reaches the outputs of the definition."""
import numpy as np
import pytest
import torch

import oracle
from paper_2503_01868_amd import binding, synth

from gpu_util import TOL, dev, draw, host, say

pytestmark = pytest.mark.gpu

# B, L, D, lh, group
SHAPES = [(1, 1, 8, 129, 8), (2, 63, 24, 9, 24), (1, 64, 72, 33, 8), (1, 65, 1000, 34, 8), (2, 129, 56, 65, 8), (1, 200, 40, 66, 8),
          (3, 300, 112, 97, 16), (1, 700, 16, 98, 16), (2, 1000, 136, 128, 8), (1, 2100, 1040, 129, 16)]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "B%dL%dD%dlh%dg%d" % s)
def test_split_products(shape, dtype):
    B, L, D, lh, group = shape
    say("split products %s %s" % (shape, dtype))
    q, k, v, h = draw(9700 + L, B, L, D, lh, group, dtype, kind="mr")
    dy = synth.normal_tensor(np.random.Generator(np.random.PCG64(9701)), (B, L, D), dtype)
    y = host(binding.hyena_mr_fwd(dev(q), dev(k), dev(v), dev(h), group))
    # fp32: a sum rounds once per 32 terms and a few times more, each 2^-24 of partial sums that are no larger than a few
    # times the result in the 2-norm, x itself and the gate 2^-24; bf16: the store, 2^-9 at most per value
    tol = 1e-6 if dtype == "f32" else 2.0 ** -8
    assert oracle.rel_err(y, oracle.gated_conv(q, k, v, h, group=group)) <= tol
    outs = binding.hyena_mr_bwd(dev(dy), dev(q), dev(k), dev(v), dev(h), group)
    ref = oracle.gated_conv_bwd(dy, q, k, v, h, group=group)
    for name, got, want in zip(("dq", "dk", "dv", "dh"), outs, ref):
        assert oracle.rel_err(host(got), want) <= (TOL["f32"] if name == "dh" else tol), name


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("group", [8, 16])
@pytest.mark.parametrize("size,tap", [(1e-18, 1.0), (1e-9, 1e-17), (1.0, 1e-35)])
def test_small_magnitudes(size, tap, group, dtype):
    """k * v, or taps, of 1e-36 and sums that are normal numbers: the same relative error as at 1."""
    say("split products, k and v of %g, taps of %g, groups of %d, %s" % (size, tap, group, dtype))
    q, k, v, h = draw(9900, 1, 300, 48, 128, group, dtype, kind="mr")
    dy = synth.normal_tensor(np.random.Generator(np.random.PCG64(9901)), (1, 300, 48), dtype)
    k, v, h = k * size, v * size, (h * np.float32(tap)).astype(np.float32)
    # gradients: the transposed sum over dy * q, times k or v (the forward's dq: times dy)
    dy, q = (dy, q) if tap < 1 else (dy * size, q * size)
    back = 1.0 if tap < 1 else 1 / size  # gates that bring the results back to sums' sizes
    tol = 1e-6 if dtype == "f32" else 2.0 ** -8
    one = torch.ones_like(q)
    y = host(binding.hyena_mr_fwd(dev(one), dev(k), dev(v), dev(h), group))
    assert oracle.rel_err(y, oracle.gated_conv(one, k, v, h, group=group)) <= tol
    kk, vv = k * back, v * back
    _, dk, dv, _ = (host(x) for x in binding.hyena_mr_bwd(dev(dy), dev(q), dev(kk), dev(vv), dev(h), group))
    _, rk, rv, _ = oracle.gated_conv_bwd(dy, q, kk, vv, h, group=group)
    assert oracle.rel_err(dk, rk) <= tol and oracle.rel_err(dv, rv) <= tol


@pytest.mark.parametrize("L,at", [(300, 0), (300, 63), (900, 640)])
def test_values_that_are_not_finite(L, at):
    B, D, lh, group = 1, 24, 128, 8
    say("split products, not finite, L=%d at=%d" % (L, at))
    q, k, v, h = draw(9800 + at, B, L, D, lh, group, "f32", kind="mr")
    dy = torch.from_numpy(np.random.Generator(np.random.PCG64(2)).standard_normal((B, L, D), dtype=np.float32))
    k[0, at, 3] = float("inf")
    k[0, at, 12], v[0, at, 12] = 3.4e38, 1.0  # finite; its bf16 head is not
    h = h.copy()
    h[1] *= np.float32(1e-2)
    h[2, 40] = np.nan
    bad = np.zeros((L, D), dtype=bool)
    bad[at:at + lh, 3] = True
    bad[40:, 16:] = True
    y = host(binding.hyena_mr_fwd(dev(q), dev(k), dev(v), dev(h), group))
    assert np.array_equal(~np.isfinite(y[0]), bad)
    with np.errstate(all="ignore"):
        ref = oracle.gated_conv(q, k, v, h, group=group)
    assert oracle.rel_err(y[0][:, 8:16], ref[0][:, 8:16]) <= 1e-6
    dq, dk, dv, _ = (host(x) for x in binding.hyena_mr_bwd(dev(dy), dev(q), dev(k), dev(v), dev(h), group))
    assert np.array_equal(~np.isfinite(dq[0]), bad)
    bad_k = np.zeros((L, D), dtype=bool)
    bad_k[:L - 40, 16:] = True
    assert np.array_equal(~np.isfinite(dk[0]), bad_k)
    bad_k[at, 3] = True  # dv = du * k
    assert np.array_equal(~np.isfinite(dv[0]), bad_k)
