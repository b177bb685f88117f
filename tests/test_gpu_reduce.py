"""The reduction of partial filter gradients: 1, 4, 32 or 256 lanes per output, by the number of outputs and of terms."""
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


def test_a_filter_shared_by_all_channels_is_no_serial_sum():
    """65536 terms of 6 outputs: 47 times the call with a filter per channel when four lanes add them, 3 to 4 times with
    256 lanes."""
    B, L, D, lh = 2, 57, 4096, 6
    x = [torch.randn((B, L, D), device="cuda:0").bfloat16() for _ in range(4)]

    def us(group):
        h = torch.randn((D // group, lh), device="cuda:0")
        times = []
        for _ in range(9):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            for _ in range(10):
                binding.hyena_se_bwd(*x, h, group)
            b.record()
            torch.cuda.synchronize()
            times.append(a.elapsed_time(b) * 100)
        return statistics.median(times)

    one, shared = us(1), us(D)
    say("hyena_se_bwd 2 x 57 x 4096: a filter per channel %.1f us, one filter %.1f us" % (one, shared))
    assert shared < 12 * one
