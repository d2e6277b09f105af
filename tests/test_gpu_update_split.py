"""GPU: fp32 updates whose generated factors are three bf16 parts each (more than 512 tiles of 32 x 32 on 256 CUs; 192 kappa and more in up to 512 tiles of
64 x 64, 512 and more beyond), at the edges of tiles, stages and the rule, against 64 bits from the library's own factors.

Bounds, u = 2^-24, s the 2-norm of an entry's terms.  f a is held to 2^-27; rounding the sum once is u sqrt(0.175) of s in the mean square, and the products left out are
u / 8; the sum walks there in as many steps as there are groups of four neighbouring kappa with a fitness, each but the first rounded at half of the size the sum has on the
way, s / sqrt(2) in the mean square: u sqrt((steps - 1) / 20) more.  So u sqrt(0.19 + (steps - 1) / 20) (2.6e-8 for a single kappa, 9.5e-8 for 192, 6.0e-7 for 8192; a
quarter on top is allowed) over all entries, in the 2-norm.  For a single entry ten times as much, of the larger of s and the
entry: the longest of a million walks are 5 s away, at their end or before it, and round at that size, and twice the deviation (7.7 is the most seen).  What the rule leaves to the fp32 chain rounds at every one of k kappa with a fitness: u (0.62 + 0.31 sqrt(k))."""
import math

import pytest

from helpers import memory_left
from paper_2511_16652_amd import binding as eb

pytestmark = pytest.mark.gpu
U = 2.0 ** -24
KEY, BEGIN = (3, 1, 9), 5


@pytest.fixture(scope="module")
def ctx():
    import torch
    c = eb.Context(0)
    yield c
    torch.cuda.synchronize()
    c.close()


def factors(ctx, begin, N, d_out, d_in, rank):
    import torch
    A, B = (torch.empty((N, d, rank), device="cuda") for d in (d_out, d_in))
    ctx.eggroll_noise_gen(eb.make_key(*KEY), eb.make_shape(begin, N, 1, d_out, d_in, rank), eb.EGG_F32, eb.EGG_NORMAL, 0, A, B)
    flat = lambda F: F.double().transpose(1, 2).reshape(N * rank, -1)  # noqa: E731
    return flat(A), flat(B)


def in_parts(d_out, d_in, K):
    t = lambda n: -(-d_out // n) * -(-d_in // n)  # noqa: E731
    return t(32) > 512 and K >= (192 if t(64) <= 512 else 512)


def unit_error(d_out, d_in, f, rank):
    import torch
    kappa = f.repeat_interleave(rank) != 0
    K, k = kappa.numel(), int(kappa.sum())
    steps = int(torch.nn.functional.pad(kappa, (0, -K % 4)).view(-1, 4).any(1).sum())
    return U * (math.sqrt(0.19 + (steps - 1) / 20) if in_parts(d_out, d_in, K) else 0.62 + 0.31 * math.sqrt(k))


def check(ctx, G, f, scale, d_out, d_in, N, rank, extra=0.0):
    import torch
    A, B = factors(ctx, BEGIN, N, d_out, d_in, rank)
    A *= f.double().repeat_interleave(rank)[:, None]
    ref = scale * (A.t().contiguous() @ B)
    s = scale * (A.square().t().contiguous() @ B.square()).sqrt()
    unit = unit_error(d_out, d_in, f, rank)
    err = (G.double() - ref).abs() - extra
    assert (err <= 10 * unit * torch.maximum(s, ref.abs())).all()
    assert err.clamp(min=0).norm() <= 1.25 * unit * s.norm()
    return ref


SHAPES = [
    (1024, 736, 191, 1), (1024, 736, 192, 1), (1024, 512, 300, 1), (1024, 520, 193, 1),     # both sides of 192 kappa and of 512 tiles
    (1032, 1022, 97, 2), (736, 1029, 50, 4), (1000, 1000, 31, 8), (1028, 741, 13, 16),       # ragged; odd widths from rank 2 on
    (2048, 1028, 511, 1), (2048, 1028, 512, 1), (1404, 2098, 1025, 1), (2052, 1026, 33, 16),  # tiles of 128, both sides of 512; the norm found beforehand
    (2048, 1024, 224, 1), (4100, 300, 8192, 1),
]


@pytest.mark.parametrize("d_out,d_in,N,rank", SHAPES)
@pytest.mark.parametrize("w", [None, "bf16", "f32"])
def test_split_update(ctx, d_out, d_in, N, rank, w):
    import torch
    g = torch.Generator("cuda").manual_seed(N)
    f = torch.randn(N, generator=g, device="cuda") * 1e-20    # (any magnitude: a power of two is taken out)
    G0 = torch.randn((d_out, d_in), generator=g, device="cuda")
    G = G0.clone()
    W0 = None if w is None else torch.randn((d_out, d_in), generator=g, device="cuda").to(torch.bfloat16 if w == "bf16" else torch.float32)
    W = None if w is None else W0.clone()
    scale, acc = 1e20, w == "f32"
    args = (eb.make_key(*KEY), eb.make_shape(BEGIN, N, 1, d_out, d_in, rank), eb.EGG_F32, f, scale, int(acc), G) + (() if w is None else (W, 0.125))
    ctx.eggroll_update(*args)
    # (the scale and the accumulation round once each)
    check(ctx, G.double() - G0.double() if acc else G, f, float(torch.tensor(scale)), d_out, d_in, N, rank, U * (G.abs() + (G - G0).abs()).double() if acc else 0.0)
    if w:
        want = W0.double() + 0.125 * G.double()
        assert ((W.double() - want).abs() <= (2.0 ** -8 if w == "bf16" else 2.0 ** -22) * (want.abs() + 1e-3)).all()


@pytest.mark.parametrize("d_out,d_in,N,rank", [(1024, 736, 192, 1), (1000, 1000, 31, 8), (2048, 1028, 700, 1), (2052, 1026, 128, 4)])
@pytest.mark.parametrize("kind", ["one", "four", "sixteen", "half small", "one large", "eight decades"])
def test_fitness_of_few_members_or_wide_range(ctx, d_out, d_in, N, rank, kind):
    """Few members with a fitness, or a range of it: what a member contributes is held to its own size wherever larger ones leave it visible.  (Half of the
    members at 1e-6 of the rest are ten times the bound on the whole; beside a single large member the entries where its term is small show the others alone.)"""
    import torch
    g = torch.Generator("cuda").manual_seed(N + 1)
    f = torch.randn(N, generator=g, device="cuda")
    few = {"one": 1, "four": 4, "sixteen": 16}.get(kind)
    if few:
        f[torch.randperm(N, generator=g, device="cuda")[few:]] = 0
    elif kind == "half small":
        f[: N // 2] *= 1e-6
    elif kind == "one large":
        f *= 1e-6
        f[N // 3] = -1.7
    else:
        f *= torch.logspace(-8, 0, N, device="cuda")
    G = torch.empty((d_out, d_in), device="cuda")
    ctx.eggroll_update(eb.make_key(*KEY), eb.make_shape(BEGIN, N, 1, d_out, d_in, rank), eb.EGG_F32, f, 1.0, 0, G)
    ref = check(ctx, G, f, 1.0, d_out, d_in, N, rank)
    if kind == "half small":   # (the bound does see those members)
        missing = torch.cat([torch.zeros_like(f[: N // 2]), f[N // 2:]])
        with pytest.raises(AssertionError):
            check(ctx, ref, missing, 1.0, d_out, d_in, N, rank)


@pytest.mark.parametrize("d_out,d_in,N,rank", [(1024, 736, 192, 1), (1000, 1000, 31, 8), (2048, 1028, 700, 1)])
@pytest.mark.parametrize("members", [1, 2, 4, None])
def test_error_is_not_larger_than_that_of_fp32_products(ctx, d_out, d_in, N, rank, members):
    """Against the update from caches, which multiplies in fp32; a single member's products are rounded at f a and at the end there, at the end alone here."""
    import torch
    errors = []
    for seed in range(4):
        g = torch.Generator("cuda").manual_seed(seed)
        f = torch.randn(N, generator=g, device="cuda")
        if members:
            f[torch.randperm(N, generator=g, device="cuda")[members:]] = 0
        key, shape = eb.make_key(*KEY), eb.make_shape(BEGIN, N, 1, d_out, d_in, rank)
        A, B = (torch.empty((N, d, rank), device="cuda") for d in (d_out, d_in))
        ctx.eggroll_noise_gen(key, shape, eb.EGG_F32, eb.EGG_NORMAL, 0, A, B)
        a, b = factors(ctx, BEGIN, N, d_out, d_in, rank)
        ref = (a * f.double().repeat_interleave(rank)[:, None]).t().contiguous() @ b
        G, Gc = (torch.empty((d_out, d_in), device="cuda") for _ in range(2))
        ctx.eggroll_update(key, shape, eb.EGG_F32, f, 1.0, 0, G)
        ctx.eggroll_update(key, shape, eb.EGG_F32, f, 1.0, 0, Gc, None, 0.0, A, B)
        errors.append([float((x.double() - ref).norm() / ref.norm()) for x in (G, Gc)])
    here, fp32 = (sum(e) for e in zip(*errors))
    assert here <= fp32


@pytest.mark.parametrize("d_out,d_in,N,rank", [(1024, 736, 192, 1), (1032, 1022, 97, 2), (2048, 1028, 512, 1), (2048, 1028, 2080, 1)])
def test_conservative_waits(ctx, d_out, d_in, N, rank):
    import torch
    f = torch.randn(N, generator=torch.Generator("cuda").manual_seed(3), device="cuda")
    outs = []
    for on in (0, 1):
        G = torch.empty((d_out, d_in), device="cuda")
        ctx.eggroll_set_conservative_waits(on)
        try:
            ctx.eggroll_update(eb.make_key(*KEY), eb.make_shape(BEGIN, N, 1, d_out, d_in, rank), eb.EGG_F32, f, 1.0, 0, G)
        finally:
            ctx.eggroll_set_conservative_waits(0)
        outs.append(G)
    assert torch.equal(*outs)


@pytest.mark.parametrize("d_out,d_in,N", [(1024, 736, 200), (2048, 1028, 600)])
@pytest.mark.parametrize("bad", [float("inf"), float("-inf"), float("nan"), "both", "large"])
def test_fitness_that_is_not_finite(ctx, bad, d_out, d_in, N):
    """An infinite fitness gives the infinities of its products, a NaN one NaN, whatever stands beside it."""
    import torch
    f = torch.randn(N, generator=torch.Generator("cuda").manual_seed(1), device="cuda")
    if bad == "both":
        f[7], f[150] = float("inf"), float("-inf")
    elif bad == "large":
        f[7], f[9] = float("inf"), 3e37   # (its entries stay finite in fp32)
    else:
        f[7] = bad
    G = torch.zeros((d_out, d_in), device="cuda")
    ctx.eggroll_update(eb.make_key(*KEY), eb.make_shape(0, N, 1, d_out, d_in, 1), eb.EGG_F32, f, 1.0, 0, G)
    A, B = factors(ctx, 0, N, d_out, d_in, 1)
    k = [i for i in range(N) if not torch.isfinite(f[i])]
    ref = sum((f[i].double() * A[i])[:, None] * B[i][None, :] for i in k)   # the terms that decide the class
    assert torch.equal(torch.isnan(G), torch.isnan(ref)) and torch.equal(torch.isposinf(G), torch.isposinf(ref)) and torch.equal(torch.isneginf(G), torch.isneginf(ref))


def test_little_memory(ctx):
    """Panels of parts take half as much again as fp32 panels: where that is not to be had the update runs from those, as before."""
    import torch
    d_out = d_in = 2048
    N = 1 << 18                                     # panels of 4.3 GB in fp32, 6.4 in parts
    f = torch.randn(N, generator=torch.Generator("cuda").manual_seed(1), device="cuda")

    def update():
        G = torch.empty((d_out, d_in), device="cuda")
        c = eb.Context(0)
        try:
            c.eggroll_update(eb.make_key(*KEY), eb.make_shape(0, N, 1, d_out, d_in, 1), eb.EGG_F32, f, 1.0, 0, G)
            torch.cuda.synchronize()
        finally:
            c.close()
        return G

    want = update()
    with memory_left(int(5.3e9)):
        got = update()
    assert not torch.equal(got, want)               # (other roundings: it was the other form)
    assert (got - want).norm() <= U * 0.31 * math.sqrt(N) * 1.5 * want.norm()
