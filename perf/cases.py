"""Performance cases of the framework: what a program that trains with EGGROLL has it do, through the binding's public calls.

Kinds of case:
  step       one ES step of one linear layer: the population's perturbed forward pass, then the update direction G
             (with `antithetic`, the members are pairs and the update runs over the pairs)
  layer      the perturbed forward pass of one layer on its way through a model: activation, residual stream
  update     the fitness-weighted update of one matrix: G, and W += lr G in place
  mlp        the GELU MLP stack, forward over all its layers
  decoder    the pre-norm decoder, tokens to logits and per-token log-likelihoods
  attention  a decoder's causal attention, with the projections for the perturbed layer that reads it
  recurrence the integer recurrent cell over its time steps
  egg        one ES step of the integer language model: forward over the tokens, log-likelihoods, update of every parameter
"""
import math

import torch

from paper_2511_16652_amd import binding as eb

_TORCH = {"f32": torch.float32, "bf16": torch.bfloat16}
_CODE = {"f32": eb.EGG_F32, "bf16": eb.EGG_BF16}
_LAYER0 = 3  # noise layer id of single-layer cases

_ctx = None


def _context():
    """The one library context that a program keeps (its scratch grows to the largest call)."""
    global _ctx
    if _ctx is None:
        _ctx = eb.Context(0)
    return _ctx


# ---- the cases ------------------------------------------------------------------------------------------------------

def listed():
    return [
        # the smallest call: a 256 x 256 fp32 layer, 64 members with one input each; launches and latency count
        {"name": "step f32 256", "kind": "step", "dtype": "f32", "d_out": 256, "d_in": 256, "members": 64, "rows": 1, "rank": 1, "antithetic": False},
        # fp32 in earnest, where a small model is trained in full precision: antithetic pairs, a few rows per member
        {"name": "step f32 2048 pairs", "kind": "step", "dtype": "f32", "d_out": 2048, "d_in": 2048, "members": 512, "rows": 4, "rank": 4, "antithetic": True},
        # an ordinary layer with a population of 4096 and one token per member (a generation step of every member)
        {"name": "step bf16 4096", "kind": "step", "dtype": "bf16", "d_out": 4096, "d_in": 4096, "members": 4096, "rows": 1, "rank": 1, "antithetic": False},
        # a small policy or adapter layer: few members, short sequences, higher rank
        {"name": "step bf16 1024 s16 r8", "kind": "step", "dtype": "bf16", "d_out": 1024, "d_in": 1024, "members": 256, "rows": 16, "rank": 8, "antithetic": False},
        # the paper's own benchmark shape, a large layer against a batch of 1024, at rank 4
        {"name": "layer 8192 b1024 r4", "kind": "layer", "dtype": "bf16", "d_out": 8192, "d_in": 8192, "members": 1024, "rows": 1, "rank": 4, "antithetic": False,
         "gelu": False, "residual": False},
        # an up-projection over sequences of ragged length (prompts of 100 tokens), an odd population
        {"name": "layer ffn s100 r2", "kind": "layer", "dtype": "bf16", "d_out": 8192, "d_in": 2048, "members": 333, "rows": 100, "rank": 2, "antithetic": False,
         "gelu": True, "residual": False},
        # the update of one matrix of the MLP stack over its whole population
        {"name": "update 8192x2048 r4", "kind": "update", "dtype": "bf16", "d_out": 8192, "d_in": 2048, "members": 16384, "rank": 4},
        # two layers of the MLP stack, 64 rows per member, rank 4
        {"name": "mlp 2x2048 s64 r4", "kind": "mlp", "d": 2048, "d_ff": 8192, "layers": 2, "members": 512, "rows": 64, "rank": 4},
        # a whole decoder call: two layers at the 1B-scale width and the full vocabulary, 256 tokens per member
        {"name": "decoder 2x2048 s256", "kind": "decoder", "d": 2048, "heads": 16, "d_ff": 8192, "vocab": 32000, "layers": 2, "members": 32, "rows": 256, "rank": 1},
        # the attention of such a decoder over a larger population
        {"name": "attention s256 hd128", "kind": "attention", "heads": 16, "head_dim": 128, "members": 512, "rows": 256},
        # the integer recurrent cell, 64 time steps of 8192 members
        {"name": "recurrence 1024 t64", "kind": "recurrence", "d": 1024, "members": 8192, "steps": 64},
        # the integer language model at its pretraining width, antithetic pairs, a few tokens per member
        {"name": "egg 256x6 t4", "kind": "egg", "d": 256, "layers": 6, "members": 32768, "tokens": 4},
    ]


def _log(rng, lo, hi, unit=1):
    """A size from lo to hi, spread over its logarithm, a multiple of `unit`."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return max(lo, min(hi, int(round(v / unit)) * unit))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "layer", "layer", "update", "mlp", "decoder", "attention", "recurrence", "egg"])
    if kind in ("step", "layer"):
        dtype = rng.choice(["bf16", "bf16", "bf16", "f32"])
        bf = dtype == "bf16"
        rank = rng.choice([1, 1, 2, 4, 8, 16])
        rows = rng.choice([1, 1, _log(rng, 2, 63), 64, 128, _log(rng, 65, 256)])
        # a power of two as often as any other multiple of the 16-byte chunk
        top = 8192 if bf else 2048
        size = lambda: rng.choice([1 << rng.randint(8, int(math.log2(top))), _log(rng, 256, top, 8)])  # noqa: E731
        d_out, d_in = size(), size()
        # rows of the call: bounded so that no drawn case costs more than the largest listed one
        most = max(rows, min(65536, int((6e11 if bf else 2e10) / (d_out * d_in))))
        members = _log(rng, 16, max(16, min(8192, most // rows)))
        anti = rng.random() < 0.3
        case = {"kind": kind, "dtype": dtype, "d_out": d_out, "d_in": d_in, "members": members + (members & 1) if anti else members, "rows": rows,
                "rank": rank, "antithetic": anti}
        if kind == "layer":
            case.update(gelu=rng.random() < 0.5, residual=rng.random() < 0.4)
        return case
    if kind == "update":
        rank = rng.choice([1, 2, 4, 8])
        return {"kind": kind, "dtype": rng.choice(["bf16", "bf16", "bf16", "f32"]), "d_out": _log(rng, 512, 4096, 8), "d_in": _log(rng, 512, 4096, 8),
                "members": _log(rng, 64, 8192 // rank), "rank": rank}
    if kind == "mlp":
        d = _log(rng, 512, 2048, 64)
        return {"kind": kind, "d": d, "d_ff": 4 * d, "layers": rng.randint(1, 2), "members": _log(rng, 32, 256), "rows": rng.choice([32, 64, 100, 128]),
                "rank": rng.choice([1, 2, 4])}
    if kind == "decoder":
        hd = rng.choice([64, 128])
        heads = rng.randint(4, 2048 // hd)
        return {"kind": kind, "d": hd * heads, "heads": heads, "d_ff": 4 * hd * heads, "vocab": _log(rng, 1000, 32000, 8), "layers": rng.randint(1, 2),
                "members": _log(rng, 8, 32), "rows": rng.choice([64, 128, 256, _log(rng, 20, 256)]), "rank": rng.choice([1, 1, 4])}
    if kind == "attention":
        return {"kind": kind, "heads": rng.randint(4, 16), "head_dim": rng.choice([32, 64, 128]), "members": _log(rng, 16, 512),
                "rows": rng.choice([64, 128, 256, _log(rng, 17, 256)])}
    if kind == "recurrence":
        return {"kind": kind, "d": _log(rng, 256, 1024, 16), "members": _log(rng, 100, 8192), "steps": _log(rng, 4, 64)}
    return {"kind": kind, "d": rng.choice([64, 256, 256]), "layers": rng.randint(1, 6), "members": 2 * _log(rng, 500, 16384), "tokens": rng.randint(1, 4)}


# ---- inputs ---------------------------------------------------------------------------------------------------------

def _gen(seed):
    return torch.Generator(device="cuda").manual_seed(int(seed))


def _normal(g, shape, std, dtype):
    return (torch.randn(shape, generator=g, device="cuda") * std).to(dtype)


def _centred(g, n):
    f = torch.randn(n, generator=g, device="cuda")
    return (f - f.mean()).contiguous()


def _int_weights(g, *shape):
    """16 N(0, 1) rounded and clipped: the initialisation of the integer model."""
    return torch.clamp(torch.round(16.0 * torch.randn(shape, generator=g, device="cuda")), -127, 127).to(torch.int8)


def _sigma(case):
    return 0.01 if case.get("dtype") == "f32" else 1e-3


_DECODER_SHAPES = lambda c: {  # noqa: E731
    "emb": (c["vocab"], c["d"]), "norm1": (c["layers"], c["d"]), "wq": (c["layers"], c["d"], c["d"]), "wk": (c["layers"], c["d"], c["d"]),
    "wv": (c["layers"], c["d"], c["d"]), "wo": (c["layers"], c["d"], c["d"]), "norm2": (c["layers"], c["d"]),
    "w_up": (c["layers"], c["d_ff"], c["d"]), "w_down": (c["layers"], c["d"], c["d_ff"]), "norm_f": (c["d"],), "head": (c["vocab"], c["d"])}


def _tensors(case, seed):
    """The inputs alone, from the seed; also what exact() starts from."""
    g, k = _gen(seed), case["kind"]
    if k in ("step", "layer"):
        dt, R = _TORCH[case["dtype"]], case["members"] * case["rows"]
        t = {"W": _normal(g, (case["d_out"], case["d_in"]), case["d_in"] ** -0.5, dt), "X": _normal(g, (R, case["d_in"]), 1.0, dt)}
        if k == "step":
            t["fitness"] = _centred(g, case["members"] // (2 if case["antithetic"] else 1))
        elif case["residual"]:
            t["R"] = _normal(g, (R, case["d_out"]), 1.0, dt)
        return t
    if k == "update":
        return {"W": _normal(g, (case["d_out"], case["d_in"]), case["d_in"] ** -0.5, _TORCH[case["dtype"]]), "fitness": _centred(g, case["members"])}
    if k == "mlp":
        L, d, ff = case["layers"], case["d"], case["d_ff"]
        return {"W1": _normal(g, (L, ff, d), d ** -0.5, torch.bfloat16), "W2": _normal(g, (L, d, ff), ff ** -0.5, torch.bfloat16),
                "X": _normal(g, (case["members"] * case["rows"], d), 1.0, torch.bfloat16)}
    if k == "decoder":
        w = {}
        for name, shape in _DECODER_SHAPES(case).items():
            if name.startswith("norm"):
                w[name] = (1.0 + 0.1 * torch.randn(shape, generator=g, device="cuda")).to(torch.bfloat16)
            else:
                w[name] = _normal(g, shape, 1.0 if name == "emb" else shape[-1] ** -0.5, torch.bfloat16)
        w["tokens"] = torch.randint(0, case["vocab"], (case["members"], case["rows"]), generator=g, device="cuda", dtype=torch.int32)
        return w
    if k == "attention":
        R, d = case["members"] * case["rows"], case["heads"] * case["head_dim"]
        return {n: _normal(g, (R, d), 1.0, torch.bfloat16) for n in ("Q", "K", "V")}
    if k == "recurrence":
        return {"W": torch.randint(-127, 128, (case["d"], case["d"]), generator=g, device="cuda", dtype=torch.int8),
                "H": torch.randint(-127, 128, (case["members"], case["d"]), generator=g, device="cuda", dtype=torch.int8)}
    D, L, N, T = case["d"], case["layers"], case["members"], case["tokens"]
    ln = lambda *s: torch.full(s, 16, dtype=torch.int8, device="cuda")  # noqa: E731
    t = {"emb": _int_weights(g, 256, D), "ln1": ln(L, D), "gru_w": _int_weights(g, L, 4, D, D), "gru_b": torch.zeros((L, 2, D), dtype=torch.int8, device="cuda"),
         "ln2": ln(L, D), "mlp1": _int_weights(g, L, 4 * D, D), "mlp2": _int_weights(g, L, D, 4 * D), "ln_out": ln(D), "head": _int_weights(g, 256, D)}
    # byte text: printable characters, frequent ones first
    p = 1.0 / (1.0 + torch.arange(95, device="cuda", dtype=torch.float32))
    text = torch.multinomial(p, (T + 1) * N, replacement=True, generator=g) + 32
    t["text"] = text.to(torch.uint8).view(T + 1, N)
    t["fitness"] = (torch.randint(0, 2, (N // 2,), generator=g, device="cuda", dtype=torch.int8) * 2 - 1).contiguous()
    return t


def prepare(case, seed):
    st = {"case": case, "ctx": _context(), **_tensors(case, seed)}
    k, rank = case["kind"], case.get("rank", 1)
    st["key"] = eb.make_key(int(seed), 1, _LAYER0)
    st["sigma"] = _sigma(case)
    new = lambda *shape, dtype: torch.empty(shape, dtype=dtype, device="cuda")  # noqa: E731
    if k in ("step", "layer"):
        st["shape"] = eb.make_shape(0, case["members"], case["rows"], case["d_out"], case["d_in"], rank, case["antithetic"])
        st["Y"] = new(case["members"] * case["rows"], case["d_out"], dtype=_TORCH[case["dtype"]])
    if k in ("step", "update"):
        ids = case["members"] // (2 if case.get("antithetic") else 1)
        st["upd_shape"] = eb.make_shape(0, ids, 1, case["d_out"], case["d_in"], rank)
        st["scale"] = eb.eggroll_default_scale(ids, st["sigma"], rank)
        st["G"] = new(case["d_out"], case["d_in"], dtype=torch.float32)
    elif k == "mlp":
        st["shape"] = eb.make_shape(0, case["members"], case["rows"], case["d"], case["d"], rank)
        st["Y"] = torch.empty_like(st["X"])
    elif k == "decoder":
        st["shape"] = eb.make_shape(0, case["members"], case["rows"], case["d"], case["d"], rank)
        st["cfg"] = eb.make_decoder_cfg(case["layers"], case["d"], case["heads"], case["d_ff"], case["vocab"])
        rows = case["members"] * case["rows"]
        st["logits"], st["loglik"] = new(rows, case["vocab"], dtype=torch.bfloat16), new(rows, dtype=torch.float32)
    elif k == "attention":
        st["O"], st["t_next"] = torch.empty_like(st["Q"]), new(case["members"] * case["rows"], dtype=torch.float32)
    elif k == "recurrence":
        st["shape"] = eb.make_shape(0, case["members"], 1, case["d"], case["d"], 1)
        st["H_out"] = torch.empty_like(st["H"])
    elif k == "egg":
        N, D, L, T = case["members"], case["d"], case["layers"], case["tokens"]
        st["shape"], st["upd_shape"] = eb.make_shape(0, N, 1, D, D, 1, True), eb.make_shape(0, N // 2, 1, D, D, 1)
        st["S"] = torch.zeros((L, N, D), dtype=torch.int8, device="cuda")
        st["S_out"], st["logits"] = torch.empty_like(st["S"]), new(T, N, 256, dtype=torch.int8)
        st["loglik"] = new(T, N, dtype=torch.int32)
        st["model"] = {n: st[n] for n in eb.EGG_MODEL_FIELDS}
        st["tokens"], st["targets"] = st["text"][:T].contiguous(), st["text"][1:].contiguous()
        st["threshold"] = eb.eggroll_int_threshold(0.2, N // 2, (8 * 9 / 3.0) ** 0.5)  # about a fifth of the entries move
    return st


# ---- one pass -------------------------------------------------------------------------------------------------------

def run(st):
    c, case, k = st["ctx"], st["case"], st["case"]["kind"]
    if k == "step":
        c.eggroll_perturbed_forward(st["key"], st["shape"], st["sigma"], eb.EGG_ACT_NONE, st["W"], st["X"], st["Y"])
        c.eggroll_update(st["key"], st["upd_shape"], _CODE[case["dtype"]], st["fitness"], st["scale"], 0, st["G"])
        return {"Y": st["Y"], "G": st["G"]}
    if k == "layer":
        act = eb.EGG_ACT_GELU if case["gelu"] else eb.EGG_ACT_NONE
        if case["residual"]:
            c.eggroll_perturbed_forward_add(st["key"], st["shape"], st["sigma"], act, st["W"], st["X"], st["R"], st["Y"])
        else:
            c.eggroll_perturbed_forward(st["key"], st["shape"], st["sigma"], act, st["W"], st["X"], st["Y"])
        return {"Y": st["Y"]}
    if k == "update":
        c.eggroll_update(st["key"], st["upd_shape"], _CODE[case["dtype"]], st["fitness"], st["scale"], 0, st["G"], st["W"], _LR)
        return {"G": st["G"], "W": st["W"]}
    if k == "mlp":
        c.eggroll_mlp_stack_forward(st["key"], st["shape"], case["layers"], case["d_ff"], st["sigma"], st["W1"], st["W2"], st["X"], st["Y"])
        return {"Y": st["Y"]}
    if k == "decoder":
        c.eggroll_decoder_forward(st["key"], st["shape"], st["cfg"], st, st["sigma"], st["tokens"], st["logits"], st["loglik"])
        return {"logits": st["logits"], "loglik": st["loglik"]}
    if k == "attention":
        c.eggroll_causal_attention_project_bf16(st["key"], 0, case["members"], case["rows"], case["heads"], case["head_dim"], st["Q"], st["K"], st["V"],
                                                st["O"], st["t_next"])
        return {"O": st["O"], "t_next": st["t_next"]}
    if k == "recurrence":
        c.eggroll_perturbed_forward_i8(st["key"], st["shape"], 8, 4, 8, case["steps"], st["W"], st["H"], st["H_out"])
        return {"H": st["H_out"]}
    N, T = case["members"], case["tokens"]
    c.eggroll_egg_forward_i8(st["key"], st["shape"], case["layers"], 8, 4, T, st["model"], st["tokens"], st["S"], st["S_out"], st["logits"])
    c.eggroll_loglik_i8(T * N, st["logits"], st["targets"], 0, st["loglik"])
    c.eggroll_egg_update_i8(st["key"], st["upd_shape"], case["layers"], 8, st["fitness"], st["threshold"], st["model"])
    return {"logits": st["logits"], "S": st["S_out"], "loglik": st["loglik"], **{n: st[n] for n in ("emb", "gru_w", "mlp1", "mlp2", "head")}}


_LR = 1e-4


# ---- what a pass cannot do without ----------------------------------------------------------------------------------

def work(case):
    k, r = case["kind"], case.get("rank", 1)
    esz = 4 if case.get("dtype") == "f32" else 2

    def layer(R, d_out, d_in):
        return 2.0 * R * d_out * d_in + 2.0 * r * R * (d_out + d_in)

    if k in ("step", "layer"):
        R, do, di = case["members"] * case["rows"], case["d_out"], case["d_in"]
        b, f = esz * (do * di + R * (do + di)), layer(R, do, di)
        if k == "step":
            ids = case["members"] // (2 if case["antithetic"] else 1)
            b, f = b + 4 * (do * di + ids), f + 2.0 * ids * r * do * di
        elif case["residual"]:
            b += esz * R * do
        return {"bytes": b, "flops": f}
    if k == "update":
        do, di, N = case["d_out"], case["d_in"], case["members"]
        return {"bytes": 4 * (do * di + N) + 2 * esz * do * di, "flops": 2.0 * N * r * do * di}
    if k == "mlp":
        R, d, ff, L = case["members"] * case["rows"], case["d"], case["d_ff"], case["layers"]
        return {"bytes": 2 * (2 * L * d * ff + 2 * R * d), "flops": L * (layer(R, ff, d) + layer(R, d, ff))}
    if k == "decoder":
        R, d, ff, V, L, S = case["members"] * case["rows"], case["d"], case["d_ff"], case["vocab"], case["layers"], case["rows"]
        att = 2.0 * R * (S + 1) * d  # half the square of scores, and as much for the values
        return {"bytes": 2 * (L * (4 * d * d + 2 * d * ff) + V * d + R * V) + 8 * R + 2 * min(R, V) * d,
                "flops": L * (4 * layer(R, d, d) + layer(R, ff, d) + layer(R, d, ff) + att) + layer(R, V, d)}
    if k == "attention":
        R, d, S = case["members"] * case["rows"], case["heads"] * case["head_dim"], case["rows"]
        return {"bytes": 2 * 4 * R * d + 4 * R, "flops": 2.0 * R * (S + 1) * d + 2.0 * R * d}
    if k == "recurrence":
        N, d, T = case["members"], case["d"], case["steps"]
        return {"bytes": d * d + 2 * N * d, "flops": T * (2.0 * N * d * d + 4.0 * N * d)}
    N, D, L, T = case["members"], case["d"], case["layers"], case["tokens"]
    params = L * 12 * D * D + 512 * D
    return {"bytes": 3 * params + T * N * (1 + 256 + 4 + 1) + 2 * L * N * D + N // 2,
            "flops": T * 2.0 * N * (L * 12 * D * D + 256 * D) + 2.0 * (N // 2) * params}


def tolerance(case):
    """Integers are the same; fp32 outputs differ by the order of sums of a few thousand terms; bf16 outputs by roundings
    of 2^-9, which in a stack of layers travel on."""
    k = case["kind"]
    if k in ("recurrence", "egg"):
        return "exact"
    if case.get("dtype") == "f32":
        return {"rel": 5e-6}
    # (against 64 bits: fp32 up to 7e-7, single bf16 layers 1.7e-3 to 1.9e-3, two MLP layers 2.2e-3, a two-layer decoder 4.5e-3)
    return {"rel": {"mlp": 9e-3, "decoder": 2e-2}.get(k, 7e-3)}


# ---- the same in 64 bits --------------------------------------------------------------------------------------------

_M32 = 0xFFFFFFFF


def _threefry(k0, k1, c0, c1):
    """Threefry-2x32-20 on 32-bit words held in int64 tensors (or ints)."""
    ks = (k0, k1, k0 ^ k1 ^ 0x1BD11BDA)
    x0, x1 = (c0 + k0) & _M32, (c1 + k1) & _M32
    for i in range(5):
        for rot in ((13, 15, 26, 6), (17, 29, 16, 24))[i % 2]:
            x0 = (x0 + x1) & _M32
            x1 = (((x1 << rot) | (x1 >> (32 - rot))) & _M32) ^ x0
        x0 = (x0 + ks[(i + 1) % 3]) & _M32
        x1 = (x1 + ks[(i + 2) % 3] + i + 1) & _M32
    return x0, x1


def _factors(seed, layer, which, members, n, dtype):
    """Entries [members][n] of the factor stream (seed, step 1, layer, which): Box-Muller in 64 bits on the stream's words,
    rounded to the type the factors are defined in."""
    k0, k1 = _threefry(int(seed) & _M32, (int(seed) >> 32) & _M32, 1, layer | (which << 31))
    out = torch.empty((members, n), dtype=torch.float64, device="cuda")
    block = torch.arange((n + 1) // 2, dtype=torch.int64, device="cuda")
    slab = max(1, (1 << 25) // block.numel())
    for lo in range(0, members, slab):
        m = torch.arange(lo, min(members, lo + slab), dtype=torch.int64, device="cuda")[:, None]
        w0, w1 = _threefry(k0, k1, block[None, :].expand(m.shape[0], -1), m)
        u1, u2 = ((w0 >> 9).double() + 0.5) * 2.0 ** -23, ((w1 >> 9).double() + 0.5) * 2.0 ** -23
        rho = torch.sqrt(-2.0 * torch.log(u1))
        z = torch.stack((rho * torch.cos(2.0 * math.pi * u2), rho * torch.sin(2.0 * math.pi * u2)), dim=-1)
        out[lo:lo + m.shape[0]] = z.view(m.shape[0], -1)[:, :n].float().to(_TORCH[dtype]).double()
    return out


def _linear(X, W, seed, layer, members, rows, rank, sigma, dtype="bf16", antithetic=False):
    """X W_i^T with W_i = W + sigma / sqrt(rank) A_i B_i^T, in 64 bits."""
    d_out, d_in = W.shape
    ids, per = (members // 2, 2 * rows) if antithetic else (members, rows)
    B = _factors(seed, layer, 1, ids, d_in * rank, dtype).view(ids, d_in, rank)
    t = torch.bmm(X.double().view(ids, per, d_in), B)
    del B
    if antithetic:
        t[:, rows:] *= -1.0
    A = _factors(seed, layer, 0, ids, d_out * rank, dtype).view(ids, d_out, rank).transpose(1, 2).contiguous()
    Y = X.double() @ W.double().t().contiguous()
    Y.view(ids, per, d_out).add_(torch.bmm(t, A), alpha=sigma / math.sqrt(rank))
    return Y


def _gelu(x):
    return 0.5 * x * (1.0 + torch.erf(x * math.sqrt(0.5)))


def _stored(x):
    """An activation between two layers is stored in bf16."""
    return x.float().to(torch.bfloat16)


def _rmsnorm(x, gain):
    x = x.double()
    return _stored(x / torch.sqrt(x.square().mean(-1, keepdim=True) + 1e-5) * gain.double())


def _attend(Q, K, V, N, S, heads):
    hd = Q.shape[1] // heads
    out = torch.empty((N * S, heads * hd), dtype=torch.float64, device="cuda")
    mask = torch.ones((S, S), dtype=torch.bool, device="cuda").triu(1)
    for lo in range(0, N, 32):
        n = min(32, N - lo)
        q, k, v = (t[lo * S:(lo + n) * S].double().view(n, S, heads, hd).transpose(1, 2).contiguous().view(n * heads, S, hd) for t in (Q, K, V))
        s = torch.bmm(q, k.transpose(1, 2).contiguous()) / math.sqrt(hd)
        s.masked_fill_(mask, float("-inf"))
        o = torch.bmm(torch.softmax(s, -1), v)
        out[lo * S:(lo + n) * S] = o.view(n, heads, S, hd).transpose(1, 2).reshape(n * S, heads * hd)
    return out


def exact(case, seed):
    k = case["kind"]
    if k in ("recurrence", "egg"):
        return None  # whole numbers: held to be the same, not near
    t, sigma, rank, dtype = _tensors(case, seed), _sigma(case), case.get("rank", 1), case.get("dtype", "bf16")
    N, S = case["members"], case.get("rows", 1)
    if k in ("step", "layer"):
        Y = _linear(t["X"], t["W"], seed, _LAYER0, N, S, rank, sigma, dtype, case["antithetic"])
        if k == "layer":
            Y = _gelu(Y) if case["gelu"] else Y
            return {"Y": Y + t["R"].double() if case["residual"] else Y}
    if k in ("step", "update"):
        ids = t["fitness"].numel()
        do, di = case["d_out"], case["d_in"]
        G = torch.zeros((do, di), dtype=torch.float64, device="cuda")
        for l0 in range(0, ids, 4096):  # the streams are addressed by member: a slab at a time would need its first id, so whole ones are cut
            if l0 == 0:
                A, B = _factors(seed, _LAYER0, 0, ids, do * rank, dtype), _factors(seed, _LAYER0, 1, ids, di * rank, dtype)
            n = min(4096, ids - l0)
            a = (A[l0:l0 + n] * t["fitness"][l0:l0 + n, None].double()).view(n, do, rank).transpose(0, 1).reshape(do, n * rank)
            b = B[l0:l0 + n].view(n, di, rank).transpose(1, 2).reshape(n * rank, di)
            G += a @ b
        G *= eb.eggroll_default_scale(ids, sigma, rank)
        return {"Y": Y, "G": G} if k == "step" else {"G": G, "W": t["W"].double() + _LR * G}
    if k == "mlp":
        h = t["X"]
        for l in range(case["layers"]):
            u = _stored(_gelu(_linear(h, t["W1"][l], seed, _LAYER0 + 2 * l, N, S, rank, sigma)))
            y = _linear(u, t["W2"][l], seed, _LAYER0 + 2 * l + 1, N, S, rank, sigma)
            h = _stored(y)
        return {"Y": y}
    if k == "attention":
        O = _attend(t["Q"], t["K"], t["V"], N, S, case["heads"])
        d = case["heads"] * case["head_dim"]
        B = _factors(seed, _LAYER0, 1, N, d, "bf16")
        return {"O": O, "t_next": torch.bmm(_stored(O).double().view(N, S, d), B.view(N, d, 1)).view(N * S)}
    x = t["emb"][t["tokens"].long().view(-1)]
    lin = lambda h, w, layer: _linear(h, w, seed, _LAYER0 + layer, N, S, rank, sigma)  # noqa: E731
    for l in range(case["layers"]):
        h = _rmsnorm(x, t["norm1"][l])
        q, kk, v = (_stored(lin(h, t[w][l], 6 * l + j)) for j, w in enumerate(("wq", "wk", "wv")))
        h = _stored(_attend(q, kk, v, N, S, case["heads"]))
        x = _stored(x.double() + lin(h, t["wo"][l], 6 * l + 3))
        u = _stored(_gelu(lin(_rmsnorm(x, t["norm2"][l]), t["w_up"][l], 6 * l + 4)))
        x = _stored(x.double() + lin(u, t["w_down"][l], 6 * l + 5))
    logits = lin(_rmsnorm(x, t["norm_f"]), t["head"], 6 * case["layers"])
    ll = torch.zeros((N, S), dtype=torch.float64, device="cuda")
    if S > 1:
        lp = _stored(logits).double().view(N, S, -1)[:, :-1]
        ll[:, :-1] = torch.gather(lp, 2, t["tokens"][:, 1:].long()[:, :, None])[:, :, 0] - torch.logsumexp(lp, -1)
    return {"logits": logits, "loglik": ll.view(-1)}
