"""Problems that do not fill the chip: the kernels cut them into tiles as short as one workgroup per compute unit makes
them, so every tile has a halo longer than itself.  Lengths around multiples of the tiles, batches, all medium paths."""
import numpy as np
import pytest

import oracle
from paper_2503_01868_amd import binding, synth

from gpu_util import TOL, check_gated, dev, draw, host, say

pytestmark = pytest.mark.gpu

SHAPES = [(1, 33, 256), (1, 130, 128), (2, 257, 256), (1, 511, 512), (1, 515, 1024), (3, 300, 256)]
LH = [9, 40, 128, 129]


@pytest.mark.parametrize("group", [16, 1])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "B%dL%dD%d" % s)
def test_medium_forward_and_gradients(shape, group):
    B, L, D = shape
    for lh in LH:
        check_gated("hyena_mr_fwd", 9500 + lh, B, L, D, lh, group, "bf16", kind="mr")
    lh = LH[L % 4]
    say("hyena_mr_bwd %s lh=%d group=%d" % (shape, lh, group))
    rng = np.random.Generator(np.random.PCG64(9600 + L))
    dy, q, k, v = (synth.normal_tensor(rng, (B, L, D), "bf16") for _ in range(4))
    h = synth.decay_filter(rng, D // group, lh)
    outs = binding.hyena_mr_bwd(dev(dy), dev(q), dev(k), dev(v), dev(h), group)
    ref = oracle.gated_conv_bwd(dy, q, k, v, h, group=group)
    for name, got, want in zip(("dq", "dk", "dv", "dh"), outs, ref):
        assert oracle.rel_err(host(got), want) <= (1e-2 if name == "dh" else TOL["bf16"]), name


@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "B%dL%dD%d" % s)
def test_chain_and_long_implicit_forward(shape):
    B, L, D = shape
    say("hyena_chain_fwd / hyena_li_fwd %s" % (shape,))
    q, k, v, h = draw(9700 + L, B, L, D, 128, 16, "bf16", kind="mr")
    rng = np.random.Generator(np.random.PCG64(9800 + L))
    hq, hk, hv = (synth.short_filter(rng, D, 7) for _ in range(3))
    y = host(binding.hyena_chain_fwd(dev(q), dev(k), dev(v), dev(hq), dev(hk), dev(hv), dev(h), 16, 1))
    assert oracle.rel_err(y, oracle.chain(q, k, v, hq, hk, hv, h, group=16, feat_group=1)) <= TOL["bf16"]
    R, lam = synth.li_params(rng, D // 16, 16)
    y = host(binding.hyena_li_fwd(dev(q), dev(k), dev(v), dev(R), dev(lam), 16))
    assert oracle.rel_err(y, oracle.li_conv(q, k, v, R, lam, group=16)) <= TOL["bf16"]
