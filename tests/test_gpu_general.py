"""The general FIR kernel (fp32, and bf16 shapes no matrix-core path takes) at the edges of its tiles: segments of 16 to 128
taps, tiles of 32 and 128 rows, walks of several tiles, 64-channel blocks with idle lanes, rows of 16-byte pieces and of
single elements; forward, gradients, featurizers; the reach of non-finite samples and taps; and what calls cost next to
their neighbours."""
import statistics

import numpy as np
import pytest
import torch

import oracle
from paper_2503_01868_amd import binding, synth

from gpu_util import TOL, check_gated, dev, draw, host, say

pytestmark = pytest.mark.gpu

# B, L, D, lh, group
SHAPES = [
    (1, 1, 1, 9, 1), (2, 31, 3, 16, 3), (1, 33, 30, 17, 1), (1, 127, 64, 63, 2), (2, 128, 65, 64, 5), (1, 129, 72, 65, 8),
    (1, 200, 40, 127, 4), (3, 300, 24, 128, 1), (1, 300, 100, 129, 20), (1, 600, 24, 192, 1), (1, 600, 24, 193, 1),
    (1, 700, 8, 257, 8), (1, 90, 16, 400, 16),
    (2, 4200, 200, 40, 8), (1, 9000, 136, 130, 1),  # a 128-row tile per workgroup; three segments in 32-row tiles
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", SHAPES, ids=lambda s: "B%dL%dD%dlh%dg%d" % s)
def test_forward(shape, dtype):
    B, L, D, lh, group = shape
    check_gated("hyena_mr_fwd", 9100 + L, B, L, D, lh, group, dtype, kind="mr")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", SHAPES[:-1], ids=lambda s: "B%dL%dD%dlh%dg%d" % s)
def test_gradients(shape, dtype):
    B, L, D, lh, group = shape
    say("hyena_mr_bwd %s %s" % (shape, dtype))
    rng = np.random.Generator(np.random.PCG64(9200 + L))
    dy, q, k, v = (synth.normal_tensor(rng, (B, L, D), dtype) for _ in range(4))
    h = synth.decay_filter(rng, D // group, lh)
    outs = binding.hyena_mr_bwd(dev(dy), dev(q), dev(k), dev(v), dev(h), group)
    ref = oracle.gated_conv_bwd(dy, q, k, v, h, group=group)
    for name, got, want in zip(("dq", "dk", "dv", "dh"), outs, ref):
        assert oracle.rel_err(host(got), want) <= (TOL["f32"] if name == "dh" else TOL[dtype]), name


@pytest.mark.parametrize("shape", [(1, 150, 6, 9, 1), (2, 513, 72, 140, 8), (1, 4500, 96, 33, 1)],
                         ids=lambda s: "B%dL%dD%dlh%dg%d" % s)
def test_ungated(shape):
    B, L, D, lh, group = shape
    say("hyena_featurize fwd/bwd %s" % (shape,))
    q, k, v, h = draw(9300 + L, B, L, D, lh, group, "f32")
    outs = binding.hyena_featurize3_fwd(dev(q), dev(k), dev(v), dev(h), dev(h), dev(h), group)
    for x, y in zip((q, k, v), outs):
        assert oracle.rel_err(host(y), oracle.causal_conv(x, h, group=group)) <= TOL["f32"]
    dx, dh = binding.hyena_featurize_bwd(dev(q), dev(k), dev(h), group)
    rx, rh = oracle.causal_conv_bwd(q, k, h, group=group)
    assert oracle.rel_err(host(dx), rx) <= TOL["f32"] and oracle.rel_err(host(dh), rh) <= TOL["f32"]


@pytest.mark.parametrize("L,at,D", [(300, 0, 16), (300, 140, 16), (300, 299, 16), (4200, 129, 16), (9000, 200, 512)])
def test_non_finite_values_reach_what_the_definition_says(L, at, D):
    """An infinite sample, and an infinite tap, make exactly those outputs non-finite whose sum has the term."""
    B, lh = 1, 128
    say("non-finite L=%d at=%d" % (L, at))
    q, k, v, h = draw(9400 + at, B, L, D, lh, 1, "f32", kind="mr")
    k[0, at, 3] = float("inf")
    h = h.copy()
    h[5, 40] = np.inf
    y = host(binding.hyena_mr_fwd(dev(q), dev(k), dev(v), dev(h), 1))
    bad = np.zeros((L, D), dtype=bool)
    bad[at:at + lh, 3] = True
    bad[40:, 5] = True
    assert np.array_equal(~np.isfinite(y[0]), bad)
    dy = torch.from_numpy(np.random.Generator(np.random.PCG64(1)).standard_normal((B, L, D), dtype=np.float32))
    dq, dk, dv, dh = (host(x) for x in binding.hyena_mr_bwd(dev(dy), dev(q), dev(k), dev(v), dev(h), 1))
    assert np.array_equal(~np.isfinite(dq[0]), bad)
    bad_k = np.zeros((L, D), dtype=bool)
    bad_k[:L - 40, 5] = True
    assert np.array_equal(~np.isfinite(dk[0]), bad_k)
    bad_k[at, 3] = True  # dv = du * k
    assert np.array_equal(~np.isfinite(dv[0]), bad_k)
    bad_h = np.zeros((D, lh), dtype=bool)
    bad_h[3, :min(lh, L - at)] = True
    assert np.array_equal(~np.isfinite(dh), bad_h)


def tile_walk(B, L, D, lh, dtype, problems):
    """(rows per tile, tiles per workgroup) of a launch with up to 128 taps, as direct_kernels.hip chooses them."""
    units = B * -(-D // 64) * problems
    single = D % (4 if dtype == "f32" else 8) != 0
    padded = 4 * 128 * -(-L // 128) > 5 * 32 * -(-L // 32)
    short_tiles = L > 128 if lh <= 32 else single and dtype == "bf16"
    rows = 128 if units * -(-L // 128) >= 256 and not padded and not short_tiles else 32
    if dtype == "bf16" and not single and lh > 32:
        rows = 32 if -(-units * -(-L // 32) // 256) == -(-units * -(-L // 64) // 256) else 64
    tiles, resident = -(-L // rows), 1024 if lh <= 32 and rows == 32 else 512

    def cost(w):
        return -(-units * w // resident) * (-(-tiles // w) + 1)

    walks, least = 1, -(-units // resident)
    for rounds in range(least, least + 4):
        w = min(rounds * resident // units, tiles)
        if cost(w) < cost(walks):
            walks = w
    return rows, -(-tiles // walks)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("D,group", [(1000, 8), (1000, 4), (1001, 1)], ids=["split", "pieces", "elements"])
@pytest.mark.parametrize("lh", [12, 20, 40, 65, 100, 128])
def test_walks_of_several_tiles(lh, D, group, dtype):
    """Walks of three tiles or more, whose halo stays in LDS: forward and gradients, on the first and the last channels.
    (Filters that 8 channels share go to the split products, but for the gradients of up to 32 taps.)"""
    B, L = 3, 5003
    for problems in (1, 2):
        rows, steps = tile_walk(B, L, D, lh, dtype, problems)
        assert steps >= 3 and rows == (32 if lh <= 32 or (dtype == "bf16" and D % 8) else 64 if dtype == "bf16" else 128)
    say("hyena_mr_fwd / bwd %d x %d x %d lh=%d group=%d %s" % (B, L, D, lh, group, dtype))
    q, k, v, h = draw(9500 + lh, B, L, D, lh, group, dtype, kind="mr")
    dy = synth.normal_tensor(np.random.Generator(np.random.PCG64(9501)), (B, L, D), dtype)
    y = host(binding.hyena_mr_fwd(dev(q), dev(k), dev(v), dev(h), group))
    grads = [host(x) for x in binding.hyena_mr_bwd(dev(dy), dev(q), dev(k), dev(v), dev(h), group)]
    for c in (slice(0, 32), slice(D - 32 - D % 8, D)):
        g = slice(c.start // group, c.stop // group)
        a = [x[..., c].contiguous() if torch.is_tensor(x) else np.ascontiguousarray(x[..., c]) for x in (dy, q, k, v)]
        f = np.ascontiguousarray(h[g])
        assert oracle.rel_err(y[..., c], oracle.gated_conv(*a[1:], f, group=group)) <= TOL[dtype]
        for name, got, want in zip(("dq", "dk", "dv", "dh"), grads, oracle.gated_conv_bwd(*a, f, group=group)):
            got = got[g] if name == "dh" else got[..., c]
            assert oracle.rel_err(got, want) <= (TOL["f32"] if name == "dh" else TOL[dtype]), name


# lh, L, D, position of the infinite sample: one segment of each length, several, more taps than steps; short and long walks
NON_FINITE = [(12, 700, 24, 40), (20, 9000, 520, 4321), (64, 300, 24, 31), (64, 9000, 520, 4500), (128, 9000, 520, 129),
              (150, 700, 24, 600), (300, 900, 24, 250), (300, 90, 24, 10)]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", NON_FINITE, ids=lambda c: "lh%dL%dD%dat%d" % c)
def test_non_finite_values_leave_the_other_outputs(case, dtype):
    """As above for every segment length and both storage types, and the outputs that stay finite are right."""
    lh, L, D, at = case
    say("non-finite %s %s" % (case, dtype))
    q, k, v, h = draw(9450 + at, 1, L, D, lh, 1, dtype, kind="mr")
    k[0, at, 3] = float("inf")
    h = h.copy()
    h[5, lh // 3] = np.inf
    dy = synth.normal_tensor(np.random.Generator(np.random.PCG64(9451)), (1, L, D), dtype)
    y = host(binding.hyena_mr_fwd(dev(q), dev(k), dev(v), dev(h), 1))
    dq, dk, dv, dh = (host(x) for x in binding.hyena_mr_bwd(dev(dy), dev(q), dev(k), dev(v), dev(h), 1))
    bad_y, bad_k = np.zeros((1, L, D), dtype=bool), np.zeros((1, L, D), dtype=bool)
    bad_y[0, at:at + lh, 3] = True
    bad_y[0, lh // 3:, 5] = True
    bad_k[0, :max(0, L - lh // 3), 5] = True
    bad_v = bad_k.copy()
    bad_v[0, at, 3] = True  # dv = du * k
    bad_h = np.zeros((D, lh), dtype=bool)
    bad_h[3, :min(lh, L - at)] = True
    ref = (oracle.gated_conv(q, k, v, h, group=1), *oracle.gated_conv_bwd(dy, q, k, v, h, group=1))
    for name, got, want, bad in zip(("y", "dq", "dk", "dv", "dh"), (y, dq, dk, dv, dh), ref, (bad_y, bad_y, bad_k, bad_v, bad_h)):
        assert np.array_equal(~np.isfinite(got), bad), name
        err = oracle.rel_err(np.where(bad, 0.0, got), np.where(bad, 0.0, np.asarray(want)))
        assert err <= (TOL["f32"] if name == "dh" else TOL[dtype]), (name, err)


def us_per_call(call):
    times = []
    for _ in range(9):
        a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
        a.record()
        for _ in range(20):
            call()
        b.record()
        torch.cuda.synchronize()
        times.append(a.elapsed_time(b) * 50)
    return statistics.median(times)


def test_odd_widths_keep_up():
    """Rows of single elements (an odd width) against rows of 16-byte pieces, 9 taps: 1.7 (fp32) and 2.1 (bf16) times as
    long with 16 rows of a workgroup's 64 channels in flight, in tiles of 128; 1.2 and 1.4 times with 32, in tiles of 32 and
    either's channel blocks together on an XCD (1.3 and 1.6 where only the even width's are)."""

    def us(D, dtype):
        x = [torch.randn((2, 1500, D), device="cuda:0").to(dtype) for _ in range(3)]
        h = torch.randn((D, 9), device="cuda:0")
        return us_per_call(lambda: binding.hyena_mr_fwd(*x, h, 1))

    for dtype in (torch.float32, torch.bfloat16):
        even, odd = us(1000, dtype), us(1001, dtype)
        say("hyena_mr_fwd 2 x 1500, 9 taps, %s: D = 1000 %.1f us, D = 1001 %.1f us" % (dtype, even, odd))
        assert odd < 1.6 * even


def test_taps_beyond_the_sequence_cost_nothing():
    """A filter longer than the sequence (history included) is one of its length: 2.2 times as long where its empty
    segments are walked through."""
    x = [torch.randn((15, 31, 333), device="cuda:0") for _ in range(3)]
    h = torch.randn((111, 800), device="cuda:0")
    short = h[:, :31].contiguous()
    a, b = (us_per_call(lambda f=f: binding.hyena_featurize3_fwd(*x, f, f, f, 3)) for f in (short, h))
    say("hyena_featurize3_fwd 15 x 31 x 333: 31 taps %.1f us, 800 taps %.1f us" % (a, b))
    assert b < 1.5 * a
    for y, z in zip(binding.hyena_featurize3_fwd(*x, short, short, short, 3), binding.hyena_featurize3_fwd(*x, h, h, h, 3)):
        assert torch.equal(y, z)
    dx = [binding.hyena_featurize_bwd(x[0], x[1], f, 3)[0] for f in (short, h)]
    assert torch.equal(*dx)


@pytest.mark.parametrize("group", [4, 8], ids=["general", "split"])
@pytest.mark.parametrize("lh", [33, 64, 65, 128])
@pytest.mark.parametrize("B,L,D", [(1, 63, 72), (2, 64, 8), (1, 65, 136), (3, 129, 200), (2, 4097, 1000), (5, 6464, 264)],
                         ids=lambda x: str(x))
def test_tiles_of_64_rows(B, L, D, lh, group):
    """bf16 rows of whole pieces go in 64-row tiles from 33 to 128 taps: a step less than a tile, one more, walks that end
    inside a tile and with one, channel blocks cut off by the width; the split products' chunks of 64 at the same sizes."""
    say("64-row tiles %d x %d x %d lh=%d group=%d" % (B, L, D, lh, group))
    q, k, v, h = draw(9600 + L + lh, B, L, D, lh, group, "bf16", kind="mr")
    dy = synth.normal_tensor(np.random.Generator(np.random.PCG64(9601)), (B, L, D), "bf16")
    y = host(binding.hyena_mr_fwd(dev(q), dev(k), dev(v), dev(h), group))
    grads = [host(x) for x in binding.hyena_mr_bwd(dev(dy), dev(q), dev(k), dev(v), dev(h), group)]
    c = slice(0, D) if D <= 264 and L < 1000 else slice(D - 24, D)  # (the last channel block where the oracle is slow)
    g = slice(c.start // group, c.stop // group)
    a = [x[..., c].contiguous() for x in (dy, q, k, v)]
    hc = np.ascontiguousarray(h[g])
    assert oracle.rel_err(y[..., c], oracle.gated_conv(*a[1:], hc, group=group)) <= TOL["bf16"]
    for name, got, want in zip(("dq", "dk", "dv", "dh"), grads, oracle.gated_conv_bwd(*a, hc, group=group)):
        got = got[g] if name == "dh" else got[..., c]
        assert oracle.rel_err(got, want) <= (TOL["f32"] if name == "dh" else TOL["bf16"]), name


# B, L, D, lh, group: more than 256 workgroups, rows that are no whole lines: one segment, several on whole and part sequences
# per XCD; of pieces and of single elements; a number of workgroups that 8 does not divide
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", [(2, 1500, 1000, 9, 1), (1, 2100, 1001, 40, 7), (5, 330, 520, 128, 4), (8, 300, 200, 250, 2),
                                  (9, 290, 203, 140, 1), (1, 2400, 504, 150, 4), (3, 200, 4090, 12, 1)],
                         ids=lambda c: "B%dL%dD%dlh%dg%d" % c)
def test_workgroups_together_on_an_xcd(case, dtype):
    B, L, D, lh, group = case
    check_gated("hyena_mr_fwd", 9700 + D, B, L, D, lh, group, dtype, kind="mr")
