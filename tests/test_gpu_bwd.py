"""GPU parity of the backward entry points against the fp64 backward oracle (itself pinned by finite
differences of the forward oracle), element by element on identical seeded inputs."""
import numpy as np
import pytest
import torch

import oracle
from paper_2503_01868_amd import binding, synth

from gpu_util import TOL, dev, host, say

pytestmark = pytest.mark.gpu

# dh is an fp32 sum over B*L*group products and is returned in fp32 for both storage types: its error is
# accumulation rounding only (~sqrt(n) * 2^-24 relative to the sum's scale for the fp32 sums inside a tile; the
# reduction over tiles and channels runs in fp64), so it is held to the fp32 bar
DH_TOL = TOL["f32"]


@pytest.fixture(autouse=True)
def _reset_options():
    yield
    for name in ("se_vec", "se_rows", "mr_rows", "mr_waves", "se_walk"):
        binding.set_option(name, 0)


def draw(seed, B, L, D, lh, group, dtype, kind):
    rng = np.random.Generator(np.random.PCG64(seed))
    dy, q, k, v = (synth.normal_tensor(rng, (B, L, D), dtype) for _ in range(4))
    n = D // group
    h = synth.short_filter(rng, n, lh) if kind == "se" else synth.decay_filter(rng, n, lh)
    return dy, q, k, v, h


def check(entry, seed, B, L, D, lh, group, dtype, kind="se", expect_ws=None):
    say("%s seed=%d B=%d L=%d D=%d lh=%d group=%d %s" % (entry, seed, B, L, D, lh, group, dtype))
    dy, q, k, v, h = draw(seed, B, L, D, lh, group, dtype, kind)
    code = binding.HY_BF16 if dtype == "bf16" else binding.HY_F32
    need = binding.lib().hyena_bwd_workspace_bytes(B, L, D, lh, group, code)
    if expect_ws is not None:
        assert (need > 0) == expect_ws
    outs = getattr(binding, entry)(dev(dy), dev(q), dev(k), dev(v), dev(h), group)
    ref = oracle.gated_conv_bwd(dy, q, k, v, h, group=group)
    for name, got, want, tol in zip(("dq", "dk", "dv", "dh"), outs, ref, (TOL[dtype],) * 3 + (DH_TOL,)):
        g = host(got)
        assert np.isfinite(g).all(), name
        err = oracle.rel_err(g, want)
        assert err <= tol, (name, err)


STENCIL_CASES = [
    (1, 1024, 256, 7, 1), (2, 777, 512, 7, 1), (3, 100, 264, 4, 1), (1, 5, 64, 7, 1), (1, 1, 8, 3, 1),
    (2, 333, 96, 1, 1), (2, 400, 128, 8, 4), (1, 300, 100, 5, 2), (2, 129, 64, 2, 64), (1, 513, 256, 3, 1),
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", STENCIL_CASES)
def test_short_filter_backward_matches_oracle(case, dtype):
    B, L, D, lh, group = case
    check("hyena_se_bwd", 71, B, L, D, lh, group, dtype, expect_ws=True)


@pytest.mark.parametrize("rows", [1, 5, 32, 1000])
def test_short_filter_backward_every_tile_length(rows):
    binding.set_option("se_rows", rows)
    for dtype in ("f32", "bf16"):
        check("hyena_se_bwd", 72, 2, 203, 192, 7, 1, dtype)


WALK_CASES = [
    # B, L, D, lh, group, se_rows (0 = the library's tile length)
    (1, 1024, 256, 7, 1, 0), (2, 777, 512, 7, 1, 128), (3, 100, 256, 4, 1, 16), (1, 5, 256, 7, 1, 0), (1, 1, 256, 3, 1, 0),
    (2, 333, 256, 1, 1, 48), (2, 400, 256, 6, 4, 80), (1, 300, 768, 5, 2, 32), (2, 129, 256, 2, 64, 0), (1, 513, 256, 3, 1, 256),
    (1, 2000, 256, 7, 256, 160),
]


@pytest.mark.parametrize("case", WALK_CASES)
def test_short_filter_backward_tile_walker_matches_oracle_and_the_stencil(case):
    """The walking kernel (`se_walk` = 1 forces it at these small sizes): against the oracle, and dq, dk, dv bit for
    bit against the stencil, whose arithmetic it repeats; dh differs only in the order of its fp32 partial sums."""
    B, L, D, lh, group, rows = case
    say("bwd walker B=%d L=%d D=%d lh=%d group=%d rows=%d" % case)
    dy, q, k, v, h = draw(80, B, L, D, lh, group, "bf16", "se")
    args = [dev(x) for x in (dy, q, k, v, h)]
    binding.set_option("se_rows", rows)
    binding.set_option("se_walk", 1)
    walked = binding.hyena_se_bwd(*args, group)
    binding.set_option("se_walk", 2)
    plain = binding.hyena_se_bwd(*args, group)
    torch.cuda.synchronize()
    for a, b in zip(walked[:3], plain[:3]):
        assert torch.equal(a, b)
    ref = oracle.gated_conv_bwd(dy, q, k, v, h, group=group)
    for name, got, want, tol in zip(("dq", "dk", "dv", "dh"), walked, ref, (TOL["bf16"],) * 3 + (DH_TOL,)):
        g = host(got)
        assert np.isfinite(g).all(), name
        assert oracle.rel_err(g, want) <= tol, name


@pytest.mark.parametrize("case", [
    (1, 300, 48, 128, 16, "bf16"), (2, 130, 64, 128, 16, "f32"), (1, 200, 40, 50, 1, "bf16"),
    (2, 150, 72, 13, 1, "f32"), (1, 90, 48, 40, 8, "bf16"), (1, 64, 33, 3, 1, "bf16"),  # odd D: general kernel
])
def test_general_backward_matches_oracle(case):
    B, L, D, lh, group, dtype = case
    check("hyena_mr_bwd", 73, B, L, D, lh, group, dtype, kind="mr")


# The matrix-core backward rounds u = k*v and g = dy*q to bf16 before the filter-gradient contraction: each
# product g*u carries two independent roundings of up to 2^-9 (rms ~1.6e-3 relative).  dh[j] sums n random-sign
# products, so its error and its own size both grow like sqrt(n): the error of an entry stays ~1.6e-3 of the
# typical |dh|; the largest of G*lh errors over the largest |dh| comes to ~2e-3..3e-3.  Bound with margin:
DH_TOL_MFMA = 1e-2

MR_BWD_CASES = [
    # B, L, D, lh, group, mr_rows
    (1, 512, 64, 128, 16, 0),
    (2, 1000, 128, 128, 16, 256),   # several tiles, halo warm-up in reversed time, ragged sequence end
    (1, 333, 64, 128, 16, 32),      # one-chunk tiles
    (2, 97, 64, 128, 16, 64),       # L < lh
    (1, 1, 64, 128, 16, 0),
    (1, 640, 192, 33, 16, 128),
    (1, 640, 64, 34, 16, 128),
    (1, 500, 64, 64, 32, 96),       # group of 32 channels: two 16-channel slices per filter
    (1, 500, 128, 65, 64, 160),
    (1, 700, 64, 129, 16, 128),
    (1, 300, 64, 9, 16, 64),        # shortest filter of this path
    (3, 256, 256, 128, 16, 128),
    (1, 2100, 128, 128, 16, 1024),
]


@pytest.mark.parametrize("case", MR_BWD_CASES)
def test_matrix_core_backward_matches_oracle(case):
    B, L, D, lh, group, rows = case
    binding.set_option("mr_rows", rows)
    say("mr bwd B=%d L=%d D=%d lh=%d group=%d rows=%d" % case)
    dy, q, k, v, h = draw(76, B, L, D, lh, group, "bf16", "mr")
    assert binding.lib().hyena_bwd_workspace_bytes(B, L, D, lh, group, binding.HY_BF16) > 0
    outs = binding.hyena_mr_bwd(dev(dy), dev(q), dev(k), dev(v), dev(h), group)
    ref = oracle.gated_conv_bwd(dy, q, k, v, h, group=group)
    for name, got, want, tol in zip(("dq", "dk", "dv", "dh"), outs, ref, (TOL["bf16"],) * 3 + (DH_TOL_MFMA,)):
        g = host(got)
        assert np.isfinite(g).all(), name
        err = oracle.rel_err(g, want)
        assert err <= tol, (name, err)


CP4_BWD_CASES = [
    # B, L, D, lh, group, mr_rows: filters not shared by 16 channels -> chunk-parallel matrix-core backward
    (1, 512, 128, 128, 1, 0),
    (2, 1000, 128, 128, 1, 256),    # several tiles: history of k, v before a tile, 3 look-ahead steps of dy, q after it
    (1, 333, 128, 100, 2, 64),      # one-iteration tiles, ragged end
    (2, 97, 128, 128, 8, 0),        # L < lh
    (1, 1, 128, 64, 1, 0),
    (1, 700, 256, 129, 1, 192),     # longest filter (nine lag blocks), tiles of three iterations
    (1, 640, 128, 9, 4, 128),       # shortest filter of this path
    (1, 450, 128, 48, 1, 64),       # three lag blocks exactly
    (1, 450, 128, 49, 1, 128),      # one tap into the fourth
    (1, 900, 384, 80, 2, 320),      # five lag blocks; tile length that is not a multiple of the ring
    (3, 260, 128, 33, 32, 0),       # groups of 32 channels through hyena_se_bwd... (see the entry chosen below)
    (1, 2100, 128, 128, 1, 1024),
]


@pytest.mark.parametrize("case", CP4_BWD_CASES)
def test_chunk_parallel_backward_matches_oracle(case):
    B, L, D, lh, group, rows = case
    binding.set_option("mr_rows", rows)
    say("cp4 bwd B=%d L=%d D=%d lh=%d group=%d rows=%d" % case)
    dy, q, k, v, h = draw(78, B, L, D, lh, group, "bf16", "mr")
    assert binding.lib().hyena_bwd_workspace_bytes(B, L, D, lh, group, binding.HY_BF16) > 0
    entry = binding.hyena_se_bwd if group == 32 else binding.hyena_mr_bwd
    # groups of 32 channels are a multiple of 16: that case runs the grouped kernel and only checks that the two
    # matrix-core paths agree on what they take
    outs = entry(dev(dy), dev(q), dev(k), dev(v), dev(h), group)
    ref = oracle.gated_conv_bwd(dy, q, k, v, h, group=group)
    for name, got, want, tol in zip(("dq", "dk", "dv", "dh"), outs, ref, (TOL["bf16"],) * 3 + (DH_TOL_MFMA,)):
        g = host(got)
        assert np.isfinite(g).all(), name
        err = oracle.rel_err(g, want)
        assert err <= tol, (name, err)


def test_chunk_parallel_backward_exact_case():
    """One filter per channel, sparse signed inputs and dyadic taps: every product and partial sum is exactly
    representable, so dq, dk, dv and dh must match the oracle bit for bit (indexing of the reversed-time launches and
    of the lag blocks of the filter gradient, through tile boundaries)."""
    B, L, D, lh, group = 2, 700, 128, 100, 1
    say("cp4 bwd exact")
    binding.set_option("mr_rows", 192)
    rng = np.random.Generator(np.random.PCG64(79))
    h = ((rng.integers(-8, 9, size=(D // group, lh)) / 8.0) * (rng.random((D // group, lh)) < 0.25)).astype(np.float32)

    def sparse(p, lo, hi):
        x = rng.integers(lo, hi + 1, (B, L, D)) * (rng.random((B, L, D)) < p)
        return torch.from_numpy(x.astype(np.float32)).bfloat16()

    dy, q, k, v = sparse(0.3, -2, 2), sparse(0.5, -1, 1), sparse(0.5, -1, 1), sparse(0.3, -1, 1)
    ref = oracle.gated_conv_bwd(dy, q, k, v, h, group=group)
    for r in ref[:3]:
        assert np.array_equal(r, torch.from_numpy(r).bfloat16().double().numpy())
    assert np.abs(ref[3]).max() < 2 ** 20 and np.array_equal(ref[3], np.round(ref[3]))
    outs = binding.hyena_mr_bwd(dev(dy), dev(q), dev(k), dev(v), dev(h), group)
    for name, got, want in zip(("dq", "dk", "dv", "dh"), outs, ref):
        assert np.array_equal(host(got), want), name


@pytest.mark.parametrize("lh", [9, 65, 66, 129])
@pytest.mark.parametrize("L,rows", [(1, 0), (3, 0), (63, 64), (64, 64), (66, 64), (126, 64), (129, 64), (192, 128), (253, 64)])
def test_chunk_parallel_backward_edges_of_tiles(L, rows, lh):
    """Ends of the sequence at every place of a 4-step piece, a 16-step group and a 64-step chunk, tiles shorter than the
    filter, both window lengths; exactly representable values, so all gradients must match bit for bit."""
    B, D, group = 2, 128, 2
    say("cp4 bwd edges L=%d rows=%d lh=%d" % (L, rows, lh))
    binding.set_option("mr_rows", rows)
    rng = np.random.Generator(np.random.PCG64(80))
    h = (rng.integers(-4, 5, size=(D // group, lh)) / 8.0 * (rng.random((D // group, lh)) < 0.3)).astype(np.float32)
    dy, q, k, v = (torch.from_numpy((rng.integers(-1, 2, (B, L, D)) * (rng.random((B, L, D)) < 0.5)).astype(np.float32)).bfloat16()
                   for _ in range(4))
    ref = oracle.gated_conv_bwd(dy, q, k, v, h, group=group)
    for r in ref[:3]:
        assert np.array_equal(r, torch.from_numpy(r).bfloat16().double().numpy())
    outs = binding.hyena_mr_bwd(dev(dy), dev(q), dev(k), dev(v), dev(h), group)
    for name, got, want in zip(("dq", "dk", "dv", "dh"), outs, ref):
        assert np.array_equal(host(got), want), name


@pytest.mark.parametrize("lh", [17, 18, 33, 34, 97, 98])
@pytest.mark.parametrize("L,rows", [(66, 64), (129, 64), (253, 64)])
def test_chunk_parallel_backward_edges_of_filters(L, rows, lh):
    """The longest and shortest filters of each number of 16-step groups."""
    test_chunk_parallel_backward_edges_of_tiles(L, rows, lh)


@pytest.mark.parametrize("lh", [9, 17, 18, 33, 34, 65, 66, 97, 98, 129])
def test_chunk_parallel_backward_reach_of_non_finite_values(lh):
    """A product spans 4 steps and multiplies its zeros, and a filter's products come in groups of 16 taps, from 34 taps on in
    pairs of groups: a NaN in u or g reaches z or du of its own channel from 3 steps on the wrong side to the end of the last
    group and 3 steps, and the filter gradient of its own filter; everything else keeps its bits."""
    B, L, D, at, c = 2, 700, 128, 400, 70
    say("cp4 bwd non-finite lh=%d" % lh)
    groups = {9: 1, 17: 1, 18: 2, 33: 2, 34: 4, 65: 4, 66: 6, 97: 6, 98: 8, 129: 8}[lh]
    dy, q, k, v, h = draw(9700 + lh, B, L, D, lh, 1, "bf16", "mr")
    clean = binding.hyena_mr_bwd(dev(dy), dev(q), dev(k), dev(v), dev(h), 1)
    span = {"u": (at, at + 16 * groups + 3), "g": (at - 16 * groups, at + 3)}
    for where, x in (("u", k), ("g", q)):
        keep = x[1, at, c].clone()
        x[1, at, c] = float("nan")
        got = binding.hyena_mr_bwd(dev(dy), dev(q), dev(k), dev(v), dev(h), 1)
        x[1, at, c] = keep
        lo, hi = span[where]
        lo -= 3
        for name, a, b in zip(("dq", "dk", "dv", "dh"), got, clean):
            a, b = a.float().cpu(), b.float().cpu()
            same = torch.ones_like(a, dtype=torch.bool)
            if name == "dh":
                same[c] = False
            else:
                same[1, lo:hi + 1, c] = False
            assert torch.equal(a[same], b[same]), (where, name)
        # what the definition makes NaN is NaN
        reach = slice(at, at + lh) if where == "u" else slice(at - lh + 1, at + 1)
        outs = (got[0],) if where == "u" else got[1:3]
        assert all(torch.isnan(o[1, reach, c]).all() for o in outs) and torch.isnan(got[3][c]).all(), where


@pytest.mark.parametrize("lh,L", [(9, 33), (128, 45)])
def test_grouped_backward_of_rows_beyond_24_bits(lh, L):
    """A row of 2^24 bytes and more and a last chunk that is not whole: wide row offsets, by the first and last channels."""
    D, group, n = 2 ** 23 + 64, 16, 64
    say("mr bwd wide rows lh=%d L=%d" % (lh, L))
    g = torch.Generator(device="cuda").manual_seed(9800 + lh)
    dy, q, k, v = (torch.randn((1, L, D), generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(4))
    h = torch.randn((D // group, lh), generator=g, device="cuda") * lh ** -0.5
    outs = binding.hyena_mr_bwd(dy, q, k, v, h, group)
    for c0 in (0, D - n):
        c = slice(c0, c0 + n)
        a = [x[..., c].cpu().contiguous() for x in (dy, q, k, v)]
        rows = slice(c0 // group, (c0 + n) // group)
        ref = oracle.gated_conv_bwd(*a, np.ascontiguousarray(h[rows].cpu().numpy()), group=group)
        for name, got, want, tol in zip(("dq", "dk", "dv", "dh"), outs, ref, (TOL["bf16"],) * 3 + (DH_TOL_MFMA,)):
            err = oracle.rel_err(host(got[rows] if name == "dh" else got[..., c]), want)
            assert err <= tol, (name, c0, err)


@pytest.mark.parametrize("lh,L", [(9, 70), (66, 130)])
def test_chunk_parallel_backward_of_rows_beyond_24_bits(lh, L):
    """A row of 2^24 bytes and more (2^23 channels and a block): the same kernel with wide row offsets, by the last channels."""
    D, group, n = 2 ** 23 + 128, 8, 64
    say("cp4 bwd wide rows lh=%d L=%d" % (lh, L))
    g = torch.Generator(device="cuda").manual_seed(9900 + lh)
    dy, q, k, v = (torch.randn((1, L, D), generator=g, device="cuda", dtype=torch.bfloat16) for _ in range(4))
    h = torch.randn((D // group, lh), generator=g, device="cuda") * lh ** -0.5
    assert binding.lib().hyena_bwd_workspace_bytes(1, L, D, lh, group, binding.HY_BF16) > 0  # (0: the general kernel)
    outs = binding.hyena_mr_bwd(dy, q, k, v, h, group)
    for c0 in (0, D - n):
        c = slice(c0, c0 + n)
        a = [x[..., c].cpu().contiguous() for x in (dy, q, k, v)]
        rows = slice(c0 // group, (c0 + n) // group)
        ref = oracle.gated_conv_bwd(*a, np.ascontiguousarray(h[rows].cpu().numpy()), group=group)
        for name, got, want, tol in zip(("dq", "dk", "dv", "dh"), outs, ref, (TOL["bf16"],) * 3 + (DH_TOL_MFMA,)):
            err = oracle.rel_err(host(got[rows] if name == "dh" else got[..., c]), want)
            assert err <= tol, (name, c0, err)


def test_matrix_core_backward_exact_case():
    """Sparse signed inputs and dyadic taps: every product and partial sum is exactly representable, so
    dq, dk, dv and dh must match the oracle bit for bit."""
    B, L, D, lh, group = 2, 700, 128, 128, 16
    say("mr bwd exact")
    binding.set_option("mr_rows", 192)
    rng = np.random.Generator(np.random.PCG64(77))
    h = ((rng.integers(-8, 9, size=(D // group, lh)) / 8.0) * (rng.random((D // group, lh)) < 0.25)).astype(np.float32)

    def sparse(p, lo, hi):
        x = rng.integers(lo, hi + 1, (B, L, D)) * (rng.random((B, L, D)) < p)
        return torch.from_numpy(x.astype(np.float32)).bfloat16()

    dy, q, k, v = sparse(0.3, -2, 2), sparse(0.5, -1, 1), sparse(0.5, -1, 1), sparse(0.3, -1, 1)
    ref = oracle.gated_conv_bwd(dy, q, k, v, h, group=group)
    for r in ref[:3]:
        assert np.array_equal(r, torch.from_numpy(r).bfloat16().double().numpy())
    assert np.abs(ref[3]).max() < 2 ** 20 and np.array_equal(ref[3], np.round(ref[3]))
    outs = binding.hyena_mr_bwd(dev(dy), dev(q), dev(k), dev(v), dev(h), group)
    for got, want in zip(outs, ref):
        assert np.array_equal(host(got), want)


def test_backward_of_a_linear_loss_equals_forward_value():
    """sum(dy * y) = sum(dq * q) = sum(dk * k) = sum(dv * v) = sum(dh * h): y is linear in each of q, k, v, h."""
    B, L, D, lh = 2, 300, 128, 7
    say("euler identity")
    dy, q, k, v, h = draw(74, B, L, D, lh, 1, "f32", "se")
    y = host(binding.hyena_se_fwd(dev(q), dev(k), dev(v), dev(h), 1))
    dq, dk, dv, dh = (host(t) for t in binding.hyena_se_bwd(dev(dy), dev(q), dev(k), dev(v), dev(h), 1))
    total = float(np.sum(dy.double().numpy() * y))
    scale = float(np.sum(np.abs(dy.double().numpy() * y)))
    for grad, arg in ((dq, q), (dk, k), (dv, v)):
        assert abs(float(np.sum(grad * arg.double().numpy())) - total) <= 1e-5 * scale
    assert abs(float(np.sum(dh * h.astype(np.float64))) - total) <= 1e-5 * scale


def test_backward_guard_bands_determinism_and_empty_batch():
    B, L, D, lh = 2, 301, 128, 7
    say("bwd guard bands")
    dy, q, k, v, h = draw(75, B, L, D, lh, 1, "bf16", "se")
    args = [dev(x) for x in (dy, q, k, v, h)]
    a = binding.hyena_se_bwd(*args, 1)
    b = binding.hyena_se_bwd(*args, 1)
    torch.cuda.synchronize()
    for x, y in zip(a, b):
        assert torch.equal(x, y)
    # L = 0: nothing to do, dh must come back as zeros
    dh = torch.full_like(args[4], 7.0)
    ptr = [t.data_ptr() for t in args[:4]] + [args[4].data_ptr()] + [t.data_ptr() for t in a[:3]] + [dh.data_ptr()]
    rc = binding.lib().hyena_se_bwd(*ptr, None, 0, B, 0, D, lh, 1, binding.HY_BF16, None)
    torch.cuda.synchronize()
    assert rc == 0 and torch.count_nonzero(dh) == 0


@pytest.mark.timeout(600)
@pytest.mark.parametrize("name", ["c1", "c2", "c2u"])
def test_backward_at_the_bench_shapes_all_outputs(name):
    """The backward workloads bench.py times (c1_bwd, c2_bwd, c2u_bwd: tile walker, one-pass matrix-core kernel,
    chunk-parallel ungrouped kernels) with bench.py's inputs and launch configuration, every element of dq, dk, dv
    and dh against the oracle."""
    w = synth.make(name)
    B, L, D, lh, group = (w[x] for x in ("B", "L", "D", "lh", "group"))
    say("backward at bench shape %s B=%d L=%d D=%d lh=%d group=%d" % (name, B, L, D, lh, group))
    rng = np.random.Generator(np.random.PCG64(synth.seed_for(name, 0) + 500000))
    dy = synth.normal_tensor(rng, (B, L, D), w["dtype"])
    entry = binding.hyena_se_bwd if w["kind"] == "se" else binding.hyena_mr_bwd
    outs = entry(dev(dy), dev(w["q"]), dev(w["k"]), dev(w["v"]), dev(w["h"]), group)
    ref = oracle.gated_conv_bwd(dy, w["q"], w["k"], w["v"], w["h"], group=group)
    dh_tol = DH_TOL if w["kind"] == "se" else DH_TOL_MFMA
    for nm, got, want, tol in zip(("dq", "dk", "dv", "dh"), outs, ref, (TOL[w["dtype"]],) * 3 + (dh_tol,)):
        g = host(got)
        assert g.shape == want.shape and np.isfinite(g).all(), nm
        err = oracle.rel_err(g, want)
        say("  %s rel_err=%.3e" % (nm, err))
        assert err <= tol, (nm, err)


@pytest.mark.timeout(600)
def test_backward_at_the_long_context_shape_on_channel_slabs():
    """c3_bwd as bench.py times it (B=1, L=131072, D=4096, lh=128, groups of 16; one-pass matrix-core kernel, four
    tiles of 32768 steps per channel block): the whole problem runs on the GPU; dq, dk, dv and the dh rows of the
    first and the last 256 channels (whole filter groups are exact sub-problems for the oracle: 100 663 296 of the
    1.6 G gradient elements, every tile boundary of those channels included) are compared element by element."""
    w = synth.make("c3")
    B, L, D, lh, group = (w[x] for x in ("B", "L", "D", "lh", "group"))
    say("backward at c3's shape B=%d L=%d D=%d lh=%d group=%d" % (B, L, D, lh, group))
    rng = np.random.Generator(np.random.PCG64(synth.seed_for("c3", 0) + 500000))
    dy = synth.normal_tensor(rng, (B, L, D), w["dtype"])
    outs = binding.hyena_mr_bwd(dev(dy), dev(w["q"]), dev(w["k"]), dev(w["v"]), dev(w["h"]), group)
    torch.cuda.synchronize()
    for c0, c1 in ((0, 256), (D - 256, D)):
        sub = [x[:, :, c0:c1].contiguous() for x in (dy, w["q"], w["k"], w["v"])]
        ref = oracle.gated_conv_bwd(*sub, w["h"][c0 // group:c1 // group], group=group)
        got = [host(o[:, :, c0:c1]) for o in outs[:3]] + [host(outs[3][c0 // group:c1 // group])]
        for nm, g, want, tol in zip(("dq", "dk", "dv", "dh"), got, ref, (TOL["bf16"],) * 3 + (DH_TOL_MFMA,)):
            assert g.shape == want.shape and np.isfinite(g).all(), nm
            err = oracle.rel_err(g, want)
            say("  channels %d..%d %s rel_err=%.3e" % (c0, c1 - 1, nm, err))
            assert err <= tol, (nm, err)


# ---------------------------------------------------------------------------------------- featurizer backward
FEAT_CASES = [
    # B, L, D, lh, group, forced tile rows (0: the library's choice)
    (1, 1024, 256, 7, 1, 0), (2, 777, 512, 7, 1, 0), (3, 100, 264, 4, 1, 0), (1, 5, 64, 7, 1, 0), (1, 1, 8, 3, 1, 0),
    (2, 333, 96, 1, 1, 0), (2, 400, 128, 8, 4, 32), (1, 300, 100, 5, 2, 1), (2, 129, 64, 2, 64, 7),
    (1, 200, 48, 20, 1, 0), (2, 150, 64, 64, 16, 0), (1, 90, 32, 128, 4, 0),     # general kernels
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", FEAT_CASES)
def test_featurizer_backward_matches_oracle(case, dtype):
    B, L, D, lh, group, rows = case
    say("hyena_featurize_bwd B=%d L=%d D=%d lh=%d group=%d rows=%d %s" % (B, L, D, lh, group, rows, dtype))
    rng = np.random.Generator(np.random.PCG64(8800 + L + lh))
    dy, x = (synth.normal_tensor(rng, (B, L, D), dtype) for _ in range(2))
    h = synth.short_filter(rng, D // group, lh) if lh <= 8 else synth.decay_filter(rng, D // group, lh)
    binding.set_option("se_rows", rows)
    code = binding.HY_BF16 if dtype == "bf16" else binding.HY_F32
    assert (binding.lib().hyena_featurize_bwd_workspace_bytes(B, L, D, lh, group, code) > 0) == (lh <= 8)
    dx, dh = binding.hyena_featurize_bwd(dev(dy), dev(x), dev(h), group)
    want_dx, want_dh = oracle.causal_conv_bwd(dy, x, h, group=group)
    gx, gh = host(dx), host(dh)
    assert np.isfinite(gx).all() and np.isfinite(gh).all()
    assert oracle.rel_err(gx, want_dx) <= TOL[dtype]
    assert oracle.rel_err(gh, want_dh) <= DH_TOL


def test_featurizer_backward_is_bit_equal_to_the_gated_backward_with_unit_gates():
    """Same kernels, same order of operations: with q = v = 1 the gated call's dk and dh are dx and dh exactly."""
    B, L, D, lh, group = 2, 600, 128, 7, 1
    rng = np.random.Generator(np.random.PCG64(8899))
    dy, x = (dev(synth.normal_tensor(rng, (B, L, D), "bf16")) for _ in range(2))
    h = dev(synth.short_filter(rng, D // group, lh))
    one = torch.ones_like(x)
    binding.set_option("se_walk", 2)   # the stencil, which is what the featurizer backward runs
    binding.set_option("se_rows", 64)  # the same tiles for both (their own choices differ at large sizes)
    _, dk, _, dh_g = binding.hyena_se_bwd(dy, one, x, one, h, group)
    dx, dh = binding.hyena_featurize_bwd(dy, x, h, group)
    assert torch.equal(dx, dk) and torch.equal(dh, dh_g)


def test_featurizer_backward_of_an_empty_batch_writes_a_zero_filter_gradient():
    h = dev(synth.short_filter(np.random.Generator(np.random.PCG64(1)), 16, 5))
    dy, x, dx = (torch.zeros((1, 10, 16), dtype=torch.bfloat16, device="cuda:0") for _ in range(3))
    dh = torch.full_like(h, 7.0)
    rc = binding.lib().hyena_featurize_bwd(dy.data_ptr(), x.data_ptr(), h.data_ptr(), dx.data_ptr(), dh.data_ptr(), None, 0,
                                           1, 0, 16, 5, 1, binding.HY_BF16, None)   # L = 0
    torch.cuda.synchronize()
    assert rc == 0 and torch.count_nonzero(dh) == 0


# ---------------------------------------------------------------------------------------- chain backward
CHAIN_BWD_CASES = [
    # B, L, D, lf, feat_group, lh, group, dtype
    (2, 700, 128, 7, 1, 128, 16, "bf16"),     # one-pass matrix-core kernel inside
    (1, 900, 128, 7, 1, 64, 1, "bf16"),       # chunk-parallel kernels inside
    (2, 500, 256, 4, 2, 7, 1, "bf16"),        # short inner filter: stencil / tile walker inside
    (1, 300, 64, 4, 1, 20, 4, "f32"),         # general kernels, fp32 throughout
    (2, 200, 48, 12, 1, 33, 2, "bf16"),       # long featurizers: general kernels for them
]


@pytest.mark.parametrize("case", CHAIN_BWD_CASES, ids=lambda c: "B%dL%dD%dlf%dfg%dlh%dg%d%s" % c)
def test_chain_backward_matches_oracle(case):
    B, L, D, lf, fg, lh, group, dtype = case
    say("hyena_chain_bwd B=%d L=%d D=%d lf=%d feat_group=%d lh=%d group=%d %s" % case)
    rng = np.random.Generator(np.random.PCG64(9100 + L + lh))
    dy, q, k, v = (synth.normal_tensor(rng, (B, L, D), dtype) for _ in range(4))
    hq, hk, hv = ((synth.short_filter if lf <= 8 else synth.decay_filter)(rng, D // fg, lf) for _ in range(3))
    h = synth.short_filter(rng, D // group, lh) if lh <= 8 else synth.decay_filter(rng, D // group, lh)
    got = binding.hyena_chain_bwd(*[dev(x) for x in (dy, q, k, v, hq, hk, hv, h)], group, fg)
    ref = oracle.chain_bwd(dy, q, k, v, hq, hk, hv, h, group=group, feat_group=fg)
    # bf16: q', k', v' and dq', dk', dv' pass through memory in bf16, so every filter gradient carries their
    # rounding like the matrix-core backward's (the same recorded bar); fp32 stays at the fp32 bar
    ftol = DH_TOL if dtype == "f32" else DH_TOL_MFMA
    for name, g, want, tol in zip(("dq", "dk", "dv", "dhq", "dhk", "dhv", "dh"), got, ref, (TOL[dtype],) * 3 + (ftol,) * 4):
        gh = host(g)
        assert gh.shape == want.shape and np.isfinite(gh).all(), name
        err = oracle.rel_err(gh, want)
        say("  %s rel_err=%.3e" % (name, err))
        assert err <= tol, (name, err)


@pytest.mark.parametrize("lh,lf", [(9, 7), (65, 1), (66, 8), (129, 5)])
@pytest.mark.parametrize("L,rows", [(1, 0), (3, 0), (31, 32), (32, 32), (34, 32), (63, 32), (129, 32), (250, 96), (517, 256)])
def test_one_pass_chain_backward_edges_of_tiles(L, rows, lh, lf):
    """Ends of the sequence at every place of a 4-step piece, a 16-step group and a 32-step chunk, tiles shorter than the inner
    filter, both window lengths, the shortest and longest featurizers, shared ones too.  The bars are the chain's (bf16 u, g,
    dq', dk', dv' and outputs: 2^-9 each, in sums of independent terms)."""
    B, D, group, fg = 2, 128, 16, 2 if lf == 5 else 1
    say("one-pass chain bwd L=%d rows=%d lh=%d lf=%d" % (L, rows, lh, lf))
    binding.set_option("mr_rows", rows)
    rng = np.random.Generator(np.random.PCG64(9300 + L + lh))
    dy, q, k, v = (synth.normal_tensor(rng, (B, L, D), "bf16") for _ in range(4))
    hq, hk, hv = (synth.short_filter(rng, D // fg, lf) for _ in range(3))
    h = synth.decay_filter(rng, D // group, lh)
    got = binding.hyena_chain_bwd(*[dev(x) for x in (dy, q, k, v, hq, hk, hv, h)], group, fg)
    ref = oracle.chain_bwd(dy, q, k, v, hq, hk, hv, h, group=group, feat_group=fg)
    for name, g, want, tol in zip(("dq", "dk", "dv", "dhq", "dhk", "dhv", "dh"), got, ref, (TOL["bf16"],) * 3 + (DH_TOL_MFMA,) * 4):
        err = oracle.rel_err(host(g), want)
        assert err <= tol, (name, err)


@pytest.mark.parametrize("lh,lf", [(9, 1), (33, 5), (65, 8), (97, 4), (129, 7)])
@pytest.mark.parametrize("L,where", [(700, 400), (700, 1), (700, 698), (64, 0), (31, 30)])
def test_one_pass_chain_backward_reach_of_non_finite_values(L, where, lh, lf):
    """A value that is not finite reaches no more of the one-pass kernel's results than of the composition's (the featurizers
    by their definition, the inner operator in whole 32-step blocks); both windows' lengths and every number of taps' quads, an
    infinite tap too.  What it does not reach keeps its bits."""
    B, D, group = 2, 128, 16
    say("one-pass chain bwd non-finite L=%d at %d lh=%d lf=%d" % (L, where, lh, lf))
    rng = np.random.Generator(np.random.PCG64(9800 + L + lh))
    dy, q, k, v = (synth.normal_tensor(rng, (B, L, D), "bf16") for _ in range(4))
    hq, hk, hv = (torch.from_numpy(synth.short_filter(rng, D, lf)) for _ in range(3))
    h = dev(synth.decay_filter(rng, D // group, lh))
    names = ("dq", "dk", "dv", "dhq", "dhk", "dhv", "dh")

    def one_pass():
        return [x.float().cpu() for x in binding.hyena_chain_bwd(*[dev(x) for x in (dy, q, k, v, hq, hk, hv)], h, group, 1)]

    def composed():
        x = [dev(t) for t in (q, k, v)]
        f = [dev(t) for t in (hq, hk, hv)]
        g = binding.hyena_mr_bwd(dev(dy), *binding.hyena_featurize3_fwd(*x, *f, 1), h, group)
        parts = [binding.hyena_featurize_bwd(gx, xx, fx, 1) for gx, xx, fx in zip(g, x, f)]
        return [p[0].float().cpu() for p in parts] + [p[1].float().cpu() for p in parts] + [g[3].float().cpu()]

    clean = one_pass()
    for bad in (float("nan"), float("inf")):
        for t, at in ((dy, (1, where, 37)), (q, (1, where, 37)), (k, (1, where, 37)), (v, (1, where, 37)), (hk, (37, lf - 1))):
            keep = t[at].clone()
            t[at] = bad
            got, want = one_pass(), composed()
            t[at] = keep
            for name, a, b, c in zip(names, got, want, clean):
                reached = ~torch.isfinite(a)
                assert not (reached & torch.isfinite(b)).any(), (name, at, bad)
                # channels of other groups, and the other batch item
                rows = a.dim() == 2
                n = a.shape[0] // (D // 16) if rows else 16  # rows or channels of a group of 16 channels
                group_of = slice(37 // 16 * n, (37 // 16 + 1) * n)
                same = torch.ones_like(a, dtype=torch.bool)
                if rows:
                    same[group_of] = False
                else:
                    same[1 if t is not hk else slice(None), :, group_of] = False
                assert torch.equal(a[same], c[same]), (name, at, bad)


@pytest.mark.timeout(900)
def test_chain_backward_at_the_chain_config_on_a_channel_slab():
    """c4_bwd as bench.py times it (B=4, L=32768, D=4096, featurizers of 7 taps, lh=128, groups of 16): the whole
    problem runs on the GPU; all seven gradients of the last 256 channels (whole filter groups and whole
    featurizer channels: an exact sub-problem for the oracle, 100 663 296 activation-gradient elements with every
    tile boundary of those channels) are compared element by element."""
    w = synth.make("c4")
    B, L, D, lh, group, lf, fg = (w[x] for x in ("B", "L", "D", "lh", "group", "lf", "feat_group"))
    say("chain backward at c4's shape B=%d L=%d D=%d lf=%d lh=%d group=%d" % (B, L, D, lf, lh, group))
    rng = np.random.Generator(np.random.PCG64(synth.seed_for("c4", 0) + 500000))
    dy = synth.normal_tensor(rng, (B, L, D), w["dtype"])
    outs = binding.hyena_chain_bwd(*[dev(x) for x in (dy, w["q"], w["k"], w["v"], w["hq"], w["hk"], w["hv"], w["h"])],
                                   group, fg)
    torch.cuda.synchronize()
    c0, c1 = D - 256, D
    sub = [x[:, :, c0:c1].contiguous() for x in (dy, w["q"], w["k"], w["v"])]
    filt = [w[n][c0 // fg:c1 // fg] for n in ("hq", "hk", "hv")] + [w["h"][c0 // group:c1 // group]]
    ref = oracle.chain_bwd(*sub, *filt, group=group, feat_group=fg)
    got = ([host(o[:, :, c0:c1]) for o in outs[:3]] + [host(o[c0 // fg:c1 // fg]) for o in outs[3:6]] +
           [host(outs[6][c0 // group:c1 // group])])
    for nm, g, want, tol in zip(("dq", "dk", "dv", "dhq", "dhk", "dhv", "dh"), got, ref,
                                (TOL["bf16"],) * 3 + (DH_TOL_MFMA,) * 4):
        assert g.shape == want.shape and np.isfinite(g).all(), nm
        err = oracle.rel_err(g, want)
        say("  channels %d..%d %s rel_err=%.3e" % (c0, c1 - 1, nm, err))
        assert err <= tol, (nm, err)


def test_chain_backward_of_an_empty_sequence_writes_zero_filter_gradients():
    rng = np.random.Generator(np.random.PCG64(2))
    hq, hk, hv = (dev(synth.short_filter(rng, 16, 5)) for _ in range(3))
    h = dev(synth.decay_filter(rng, 4, 20))
    t = [torch.zeros((1, 10, 16), dtype=torch.bfloat16, device="cuda:0") for _ in range(7)]
    grads = [torch.full_like(f, 7.0) for f in (hq, hk, hv, h)]
    ptrs = [x.data_ptr() for x in t[:4] + [hq, hk, hv, h] + t[4:] + grads]
    rc = binding.lib().hyena_chain_bwd(*ptrs, None, 0, 1, 0, 16, 5, 1, 20, 4, binding.HY_BF16, None)   # L = 0
    torch.cuda.synchronize()
    assert rc == 0 and all(torch.count_nonzero(g) == 0 for g in grads)
