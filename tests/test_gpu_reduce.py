"""The reductions of partial filter gradients: 1, 4, 32 or 256 lanes per output, by the number of outputs and of terms."""
import statistics

import numpy as np
import pytest
import torch

import oracle
from paper_2503_01868_amd import binding, synth

from gpu_util import TOL, dev, host, say

pytestmark = pytest.mark.gpu

# L, D, lh, group with tiles of 8 steps: D / group * lh outputs of L / 8 * group terms
CASES = [
    (64, 64, 7, 1), (65, 64, 7, 1),            # 8 and 9 terms
    (2048, 64, 7, 1), (2049, 64, 7, 1),        # 256 and 257 terms of 448 outputs
    (2048, 64, 7, 16), (2049, 64, 7, 16),      # 4096 and 4112 terms of 28 outputs
    (32832, 74, 7, 1),                         # 4104 terms of 518 outputs
    (2056, 1024, 8, 1), (2056, 1025, 8, 1),    # 257 terms of 8192 and 8200 outputs
    (100, 48, 1, 48),                          # one output
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "L%dD%dlh%dg%d" % c)
def test_filter_gradient(case):
    L, D, lh, group = case
    say("hyena_featurize_bwd %s, tiles of 8 steps" % (case,))
    rng = np.random.Generator(np.random.PCG64(9900 + L))
    dy, x = (synth.normal_tensor(rng, (1, L, D), "f32") for _ in range(2))
    h = synth.short_filter(rng, D // group, lh)
    binding.set_option("se_rows", 8)
    try:
        dx, dh = binding.hyena_featurize_bwd(dev(dy), dev(x), dev(h), group)
    finally:
        binding.set_option("se_rows", 0)
    rx, rh = oracle.causal_conv_bwd(dy, x, h, group=group)
    assert oracle.rel_err(host(dx), rx) <= TOL["f32"] and oracle.rel_err(host(dh), rh) <= TOL["f32"]


def us_per_call(call):
    times = []
    for _ in range(9):
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        for _ in range(10):
            call()
        b.record()
        torch.cuda.synchronize()
        times.append(a.elapsed_time(b) * 100)
    return statistics.median(times)


def test_a_filter_shared_by_all_channels_is_no_serial_sum():
    """65536 terms of 6 outputs: 47 times the call with a filter per channel when four lanes add them, 3 to 4 times with
    256 lanes."""
    B, L, D, lh = 2, 57, 4096, 6
    x = [torch.randn((B, L, D), device="cuda:0").bfloat16() for _ in range(4)]

    one, shared = (us_per_call(lambda h=torch.randn((D // g, lh), device="cuda:0"), g=g: binding.hyena_se_bwd(*x, h, g))
                   for g in (1, D))
    say("hyena_se_bwd 2 x 57 x 4096: a filter per channel %.1f us, one filter %.1f us" % (one, shared))
    assert shared < 12 * one


# B, L, D, lh, group on the general path, whose tiles of time leave B * tiles * (the group's odd part) terms per output
TILED = [(8, 43, 333, 12, 333), (2, 700, 36, 40, 9), (3, 130, 600, 9, 75), (1, 2100, 7, 20, 7), (5, 64, 260, 17, 65)]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", TILED, ids=lambda c: "B%dL%dD%dlh%dg%d" % c)
def test_filter_gradient_of_the_general_path(case, dtype):
    B, L, D, lh, group = case
    say("hyena_mr_bwd %s %s" % (case, dtype))
    rng = np.random.Generator(np.random.PCG64(9950 + L))
    dy, q, k, v = (synth.normal_tensor(rng, (B, L, D), dtype) for _ in range(4))
    h = synth.decay_filter(rng, D // group, lh)
    dh = binding.hyena_mr_bwd(dev(dy), dev(q), dev(k), dev(v), dev(h), group)[3]
    assert oracle.rel_err(host(dh), oracle.gated_conv_bwd(dy, q, k, v, h, group=group)[3]) <= TOL["f32"]


def test_a_general_filter_shared_by_all_channels_is_no_serial_sum():
    """2664 terms of 12 outputs: 21 times the call with a filter per channel when a lane walks each tile's rows alone, about
    as long with 32 lanes."""
    B, L, D, lh = 8, 43, 333, 12
    x = [torch.randn((B, L, D), device="cuda:0") for _ in range(4)]
    one, shared = (us_per_call(lambda h=torch.randn((D // g, lh), device="cuda:0"), g=g: binding.hyena_mr_bwd(*x, h, g))
                   for g in (1, D))
    say("hyena_mr_bwd 8 x 43 x 333: a filter per channel %.1f us, one filter %.1f us" % (one, shared))
    assert shared < 5 * one


def test_tiny_filter_gradients_stay_short():
    """85 steps of 72 channels in one filter of 100 taps: 2.4 times the call with 8 steps when two workgroups walk them in
    tiles, 1.2 times when a workgroup per tap sums them."""

    def call(L):
        x = [torch.randn((1, L, 72), device="cuda:0") for _ in range(4)]
        h = torch.randn((1, 100), device="cuda:0")
        return us_per_call(lambda: binding.hyena_mr_bwd(*x, h, 72))

    short, long = call(8), call(85)
    say("hyena_mr_bwd 1 x L x 72, 100 taps: L = 8 %.1f us, L = 85 %.1f us" % (short, long))
    assert long < 1.8 * short
