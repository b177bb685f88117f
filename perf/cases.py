"""Performance cases of the Hyena operators: the calls a program makes, over the range of sizes it makes them with.

A case names an operator, its shape ``B, L, D``, its filters and its storage type:

* ``se_fwd`` / ``se_bwd``: Hyena-SE (short filters, one per channel), forward and gradients;
* ``mr_fwd`` / ``mr_bwd``: Hyena-MR (medium filters; ``group`` channels share one), forward and gradients;
* ``mr_train``: Hyena-MR forward and then its gradients, what a training step asks of the operator;
* ``li_fwd``: Hyena-LI (the filter is a sum of ``order`` exponentials as long as the sequence);
* ``chain_fwd`` / ``chain_bwd``: featurizer convolutions on q, k, v and the Hyena-MR operator on their results.

Inputs follow the recipe of ``paper_2503_01868_amd.synth`` (activations N(0, 1); short filters N(0, 1/lh); medium
filters with an exponential decay drawn per filter; poles with time constants from one step to a thousand), drawn on
the GPU from the seed alone.
"""
import math

import torch

import paper_2503_01868_amd as hy

DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}
BACKWARD = ("se_bwd", "mr_bwd", "mr_train", "chain_bwd")


def listed():
    return [
        # the smallest configuration of the repository (fp32, one filter per channel): a call whose latency is what counts
        dict(name="se_fwd_f32_tiny", op="se_fwd", B=1, L=1024, D=256, lh=7, group=1, dtype="f32"),
        # Hyena-SE prefill at the width of the 7B models, context 8K
        dict(name="se_fwd", op="se_fwd", B=1, L=8192, D=4096, lh=7, group=1, dtype="bf16"),
        # Hyena-MR prefill of a long context (128K)
        dict(name="mr_fwd_long", op="mr_fwd", B=1, L=131072, D=4096, lh=128, group=16, dtype="bf16"),
        # a ragged batch of a model whose width and group do not tile a matrix core
        dict(name="mr_fwd_ragged", op="mr_fwd", B=3, L=5003, D=1000, lh=128, group=8, dtype="bf16"),
        # Hyena-MR with one filter per channel, context 8K
        dict(name="mr_fwd_ungrouped", op="mr_fwd", B=1, L=8192, D=4096, lh=128, group=1, dtype="bf16"),
        # Hyena-LI prefill, context 8K
        dict(name="li_fwd", op="li_fwd", B=1, L=8192, D=4096, order=16, group=16, dtype="bf16"),
        # the whole operator on a batch of long sequences
        dict(name="chain_fwd", op="chain_fwd", B=4, L=32768, D=4096, lf=7, feat_group=1, lh=128, group=16, dtype="bf16"),
        # gradients of the whole operator for one training sequence
        dict(name="chain_bwd", op="chain_bwd", B=1, L=8192, D=4096, lf=7, feat_group=1, lh=128, group=16, dtype="bf16"),
        # gradients of Hyena-SE for one training sequence
        dict(name="se_bwd", op="se_bwd", B=1, L=8192, D=4096, lh=7, group=1, dtype="bf16"),
        # gradients of Hyena-MR for a batch that is no power of two, of sequences that are no multiple of a tile
        dict(name="mr_bwd", op="mr_bwd", B=3, L=5000, D=2048, lh=128, group=16, dtype="bf16"),
        # gradients of Hyena-MR with one filter per channel
        dict(name="mr_bwd_ungrouped", op="mr_bwd", B=1, L=8192, D=4096, lh=128, group=1, dtype="bf16"),
        # a training step of Hyena-MR in full precision (small models, reference runs)
        dict(name="mr_train_f32", op="mr_train", B=2, L=2048, D=1024, lh=128, group=16, dtype="f32"),
    ]


def _between(rng, lo, hi):
    """A whole number, uniform in its logarithm."""
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["se_fwd_f32", "se_fwd", "mr_fwd", "mr_fwd_ungrouped", "li_fwd", "chain_fwd", "chain_bwd", "se_bwd",
                       "mr_bwd", "mr_bwd_ungrouped", "mr_train_f32"])
    dtype = "f32" if kind.endswith("_f32") else "bf16"
    op = kind.replace("_f32", "").replace("_ungrouped", "")
    D = rng.choice([256, 512, 768, 1000, 1024, 1536, 2048, 2560, 4096])
    case = dict(op=op, B=1, L=1, D=D, dtype=dtype)
    if op.startswith("se"):
        case.update(lh=rng.randint(4, 7), group=1)
    elif op == "li_fwd":
        case.update(D=D if D % 16 == 0 else 1024, order=rng.randint(4, 16), group=16)
    else:
        group = rng.choice([1, 2, 4, 8]) if D % 16 or kind.endswith("_ungrouped") else 16
        case.update(lh=rng.choice([rng.randint(16, 128), 128]), group=group)
        if op.startswith("chain"):
            case.update(lf=rng.randint(4, 7), feat_group=1)
    # elements of one activation tensor: from a few hundred steps of a narrow model to what the listed cases hold
    most = 2 ** 22 if op == "mr_train" or (op not in ("se_fwd", "se_bwd") and D % 16) else 2 ** 25 if op in BACKWARD else 2 ** 27
    tokens = _between(rng, 512, most // case["D"])
    case["B"] = min(_between(rng, 1, 6), max(1, tokens // 256))
    case["L"] = tokens // case["B"]
    return case


def prepare(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    B, L, D = case["B"], case["L"], case["D"]

    def normal(*shape, dtype=torch.float32):
        return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32).to(dtype)

    def short(n, taps):
        return normal(n, taps) * taps ** -0.5

    def decaying(n, taps):
        alpha = 0.01 + 0.09 * torch.rand((n, 1), generator=g, device="cuda")
        return short(n, taps) * torch.exp(-alpha * torch.arange(taps, device="cuda"))

    state = dict(case)
    for name in ("q", "k", "v") + (("dy",) if case["op"] in BACKWARD else ()):
        state[name] = normal(B, L, D, dtype=DTYPES[case["dtype"]])
    n = D // case["group"]
    if case["op"] == "li_fwd":
        state["R"] = normal(n, case["order"]) * case["order"] ** -0.5
        a = torch.rand((n, case["order"]), generator=g, device="cuda") * math.log(1e3) + math.log(1e-3)
        state["lam"] = torch.exp(-torch.exp(a))
    else:
        state["h"] = short(n, case["lh"]) if case["op"].startswith("se") else decaying(n, case["lh"])
    if case["op"].startswith("chain"):
        for name in ("hq", "hk", "hv"):
            state[name] = short(D // case["feat_group"], case["lf"])
    return state


def run(s):
    op = s["op"]
    if op == "se_fwd":
        return hy.hyena_se_fwd(s["q"], s["k"], s["v"], s["h"], s["group"])
    if op == "mr_fwd":
        return hy.hyena_mr_fwd(s["q"], s["k"], s["v"], s["h"], s["group"])
    if op == "li_fwd":
        return hy.hyena_li_fwd(s["q"], s["k"], s["v"], s["R"], s["lam"], s["group"])
    if op == "chain_fwd":
        return hy.hyena_chain_fwd(s["q"], s["k"], s["v"], s["hq"], s["hk"], s["hv"], s["h"], s["group"], s["feat_group"])
    if op == "chain_bwd":
        names = ("dq", "dk", "dv", "dhq", "dhk", "dhv", "dh")
        return dict(zip(names, hy.hyena_chain_bwd(s["dy"], s["q"], s["k"], s["v"], s["hq"], s["hk"], s["hv"], s["h"],
                                                  s["group"], s["feat_group"])))
    if op == "se_bwd":
        return dict(zip(("dq", "dk", "dv", "dh"), hy.hyena_se_bwd(s["dy"], s["q"], s["k"], s["v"], s["h"], s["group"])))
    if op == "mr_bwd":
        return dict(zip(("dq", "dk", "dv", "dh"), hy.hyena_mr_bwd(s["dy"], s["q"], s["k"], s["v"], s["h"], s["group"])))
    y = hy.hyena_mr_fwd(s["q"], s["k"], s["v"], s["h"], s["group"])
    out = dict(zip(("dq", "dk", "dv", "dh"), hy.hyena_mr_bwd(s["dy"], s["q"], s["k"], s["v"], s["h"], s["group"])))
    out["y"] = y
    return out


def work(case):
    op, n = case["op"], case["B"] * case["L"] * case["D"]
    size = 4 if case["dtype"] == "f32" else 2
    tensors = {"mr_train": 8}.get(op, 7 if op in BACKWARD else 4)
    rows = case["D"] // case["group"]
    if op == "li_fwd":  # the recurrent form: advance and read `order` running sums
        return {"bytes": tensors * n * size + 8 * rows * case["order"], "flops": n * (4 * case["order"] + 2)}
    table, taps = 4 * rows * case["lh"], 2 * case["lh"]
    flops = {"se_fwd": taps + 2, "mr_fwd": taps + 2, "se_bwd": 3 * taps + 5, "mr_bwd": 3 * taps + 5, "mr_train": 3 * taps + 6,
             "chain_fwd": taps + 2, "chain_bwd": 3 * taps + 5}[op]
    if op.startswith("chain"):
        table += 12 * case["D"] // case["feat_group"] * case["lf"]
        flops += 3 * 2 * case["lf"] * (3 if op == "chain_bwd" else 1)
    return {"bytes": tensors * n * size + table * (2 if op in BACKWARD else 1), "flops": n * flops}


def tolerance(case):
    """Four times what the outputs measure against ``exact``."""
    if case["dtype"] == "f32":
        return {"rel": 2e-6}
    # one rounding to bf16 at the store on the short filters; u and the filter enter the matrix products rounded to
    # bf16 on the medium ones; the chain's gradients also pass through memory in bf16 between its steps
    return {"rel": {"se_fwd": 7e-3, "se_bwd": 7e-3, "chain_bwd": 1.6e-2}.get(case["op"], 1.2e-2)}


# ---- the same outputs in 64 bits, slab by slab of channels (a channel depends on no other, apart from the filter
# gradients, which sum over the channels of a group; slabs hold whole groups)


def _conv(h, x):
    """sum_j h[c, j] x[b, t - j, c] for x [B, L, C], h [C, taps]."""
    z = x * h[:, 0]
    for j in range(1, min(h.shape[1], x.shape[1])):
        z[:, j:].addcmul_(x[:, :-j], h[:, j].expand_as(x[:, :-j]))
    return z


def _conv_t(h, x):
    """sum_j h[c, j] x[b, t + j, c]."""
    z = x * h[:, 0]
    for j in range(1, min(h.shape[1], x.shape[1])):
        z[:, :-j].addcmul_(x[:, j:], h[:, j].expand_as(x[:, j:]))
    return z


def _correlate(y, x, taps, group):
    """sum over b, t and the channels of a group of y[b, t, c] x[b, t - j, c]: [C // group, taps]."""
    L, C = x.shape[1], x.shape[2]
    d = torch.zeros((C, taps), dtype=torch.float64, device=x.device)
    for j in range(min(taps, L)):
        d[:, j] = (y[:, j:] * x[:, :L - j]).sum(dim=(0, 1))
    return d.view(C // group, group, taps).sum(dim=1)


def _inner_bwd(dy, q, k, v, hc, taps, group):
    u, g = k * v, dy * q
    du = _conv_t(hc, g)
    return dy * _conv(hc, u), du * v, du * k, _correlate(g, u, taps, group)


def _long(u, R, lam):
    """sum_j (sum_n R[g, n] lam[g, n]^j) u[t - j] in its recurrent form, in chunks; u [B, L, G * group]."""
    B, L, D = u.shape
    G, order = R.shape
    T = 256
    t = torch.arange(T, device=u.device, dtype=torch.float64)
    powers = lam[:, :, None] ** t  # [G, order, T]
    taps = (R[:, :, None] * powers).sum(dim=1)  # [G, T]
    lag = (t[:, None] - t[None, :]).long()
    toeplitz = torch.where(lag >= 0, taps[:, lag.clamp(min=0)], torch.zeros((), dtype=torch.float64, device=u.device))
    read = (R[:, :, None] * powers * lam[:, :, None]).transpose(1, 2).contiguous()  # state before a chunk -> its outputs
    feed = powers.flip(2).contiguous()  # a chunk's inputs -> state after it
    z = torch.empty_like(u)
    s = torch.zeros((G, order, B * (D // G)), dtype=torch.float64, device=u.device)
    for t0 in range(0, L, T):
        x = u[:, t0:t0 + T]
        m = x.shape[1]
        x = x.reshape(B, m, G, D // G).permute(2, 1, 0, 3).reshape(G, m, -1)
        o = torch.bmm(toeplitz[:, :m, :m].contiguous(), x) + torch.bmm(read[:, :m].contiguous(), s)
        z[:, t0:t0 + T] = o.view(G, m, B, D // G).permute(2, 1, 0, 3).reshape(B, m, D)
        if m == T:
            s = s * (lam ** T)[:, :, None] + torch.bmm(feed, x)
    return z


def _exact_slab(s, op, c0, c1):
    def wide(name):
        return s[name][:, :, c0:c1].double()

    def per_channel(name, group):
        return s[name][c0 // group:c1 // group].double().repeat_interleave(group, dim=0)

    q, k, v = wide("q"), wide("k"), wide("v")
    group = s["group"]
    if op == "li_fwd":
        rows = slice(c0 // group, c1 // group)
        return {"y": q * _long(k * v, s["R"][rows].double(), s["lam"][rows].double())}
    h = per_channel("h", group)
    if op.startswith("chain"):
        hq, hk, hv = (per_channel(n, s["feat_group"]) for n in ("hq", "hk", "hv"))
        fq, fk, fv = _conv(hq, q), _conv(hk, k), _conv(hv, v)
        if op == "chain_fwd":
            return {"y": fq * _conv(h, fk * fv)}
        gq, gk, gv, dh = _inner_bwd(wide("dy"), fq, fk, fv, h, s["lh"], group)
        out = {"dh": dh}
        for name, g, x, f in (("q", gq, q, hq), ("k", gk, k, hk), ("v", gv, v, hv)):
            out["d" + name] = _conv_t(f, g)
            out["dh" + name] = _correlate(g, x, s["lf"], s["feat_group"])
        return out
    out = {} if op in ("se_bwd", "mr_bwd") else {"y": q * _conv(h, k * v)}
    if op in BACKWARD:
        out.update(zip(("dq", "dk", "dv", "dh"), _inner_bwd(wide("dy"), q, k, v, h, s["lh"], group)))
    return out


def exact(case, seed):
    s = prepare(case, seed)
    D = case["D"]
    unit = math.lcm(case["group"], case.get("feat_group", 1))
    step = max(unit, 2 ** 26 // (case["B"] * case["L"]) // unit * unit)  # 0.5 GiB per tensor of a slab
    whole = {}
    for c0 in range(0, D, step):
        c1 = min(D, c0 + step)
        for name, x in _exact_slab(s, case["op"], c0, c1).items():
            if x.dim() == 3:
                if name not in whole:
                    whole[name] = torch.empty((x.shape[0], x.shape[1], D), dtype=torch.float64, device=x.device)
                whole[name][:, :, c0:c1] = x
            else:
                whole.setdefault(name, []).append(x)
    whole = {name: torch.cat(x) if isinstance(x, list) else x for name, x in whole.items()}
    return whole if case["op"] in BACKWARD else whole["y"]
