"""Hyena-MR gradients of a batch: tiles that run on from one batch item into the next give every item the bits of a call of
its own, and filter gradients that add up."""
import numpy as np
import pytest
import torch

import oracle
from paper_2503_01868_amd import binding, synth

from gpu_util import dev, draw, say

pytestmark = pytest.mark.gpu

# B, L, D, lh: batches whose tiles run on from one item into the next (the first six; tiles that begin between two items,
# in an item's last chunk, in its middle); others that do not divide 256 workgroups; items of one chunk of 32
# steps, of a chunk and a step, of a chunk less a step, shorter than the filter, of many tiles; filters of 2 to 5 source blocks
CASES = [(3, 250, 8192, 128), (5, 70, 4096, 33), (3, 129, 8192, 129), (257, 40, 64, 30), (3, 5000, 2048, 128), (5, 1000, 4096, 70),
         (3, 1000, 2048, 128), (5, 33, 1536, 129), (7, 31, 192, 40), (2, 32, 64, 65), (6, 65, 768, 97),
         (3, 2500, 64, 9), (5, 1, 128, 128)]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "B%dL%dD%dlh%d" % c)
def test_items_have_the_bits_of_their_own_calls(case):
    B, L, D, lh = case
    say("hyena_mr_bwd batch %s" % (case,))
    q, k, v, h = draw(9950 + L, B, L, D, lh, 16, "bf16", kind="mr")
    dy = synth.normal_tensor(np.random.Generator(np.random.PCG64(9951)), (B, L, D), "bf16")
    t = [dev(x) for x in (dy, q, k, v)]
    hd = dev(h)
    whole = binding.hyena_mr_bwd(*t, hd, 16)
    dh = torch.zeros((D // 16, lh), dtype=torch.float64, device="cuda:0")
    for b in range(B):
        own = binding.hyena_mr_bwd(*(x[b:b + 1].contiguous() for x in t), hd, 16)
        for name, x, y in zip(("dq", "dk", "dv"), whole, own):
            assert torch.equal(x[b], y[0]), (name, b)
        dh += own[3].double()
    # fp32 partial sums of other stretches of time on either side
    assert oracle.rel_err(whole[3].double().cpu().numpy(), dh.cpu().numpy()) <= 1e-5
