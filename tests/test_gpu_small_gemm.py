"""GPU: products too small for the chip-filling tiles (fp32 updates: 32 and 64 tiles with K split over four waves; bf16 updates and layers: 32 and 64 tiles,
and one 128 x 128 tile per CU, with four stages in flight; fp32 layers: 32 tiles with four stages in flight), at the edges of their
K ranges and of the rule between them, and the tiles that follow them.

References in 64 bits from the library's own factors; fp32: 1e-5 of |value| + rms (sums of up to 2064 products in another order);
bf16 outputs: one rounding, 2^-8; update panels in fp16: 2^-11 per term, random sign, so 2e-3 of the rms covers every entry."""
import math

import pytest

from paper_2511_16652_amd import binding as eb

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    import torch
    c = eb.Context(0)
    yield c
    torch.cuda.synchronize()
    c.close()


def factors(ctx, key, ids, n, rank, which, tdt, code):
    import torch
    F = torch.empty((ids, n, rank), dtype=tdt, device="cuda")
    shape = eb.make_shape(0, ids, 1, n, n, rank)
    ctx.eggroll_noise_gen(key, shape, code, eb.EGG_NORMAL, 0, *((F, None) if which == 0 else (None, F)))
    return F


@pytest.mark.parametrize("dtype,d_out,d_in,N,S,rank,cache", [
    ("f32", 4, 4, 1, 1, 1, 0), ("f32", 36, 12, 33, 1, 1, 1), ("f32", 100, 68, 9, 3, 4, 0), ("f32", 256, 2064, 5, 7, 2, 0),
    ("f32", 1028, 132, 260, 2, 1, 0),       # 33 x 17 tiles of 32
    ("bf16", 4, 8, 1, 1, 1, 0), ("bf16", 36, 24, 33, 1, 1, 1), ("bf16", 100, 520, 9, 3, 4, 0), ("bf16", 132, 2056, 5, 7, 16, 0),
    ("bf16", 520, 64, 33, 16, 2, 0),        # 17 x 17 tiles of 32
    ("bf16", 1028, 64, 33, 16, 2, 0),       # 33 x 17 of them, 17 x 9 of 64; one stage of K
    ("bf16", 1028, 136, 33, 16, 4, 0), ("bf16", 1028, 200, 33, 16, 8, 0), ("bf16", 1028, 256, 33, 16, 1, 0),   # two, three and four stages
    ("bf16", 1028, 512, 550, 2, 1, 1), ("bf16", 4100, 64, 1025, 2, 1, 1), ("bf16", 4100, 64, 2050, 1, 4, 0), ("bf16", 4100, 64, 2050, 1, 8, 1),   # past them all, fewer
    ("bf16", 4100, 72, 683, 3, 16, 0), ("bf16", 3076, 64, 4100, 1, 8, 0), ("bf16", 3076, 72, 1367, 3, 16, 0),   # than 15 rows: 128, 256 x 128 and 256 tiles
    ("bf16", 1028, 328, 33, 16, 1, 0), ("bf16", 1028, 392, 33, 16, 1, 0), ("bf16", 1028, 456, 33, 16, 1, 0),   # five, six, seven
])
def test_small_forward(ctx, dtype, d_out, d_in, N, S, rank, cache):
    import torch
    tdt, code = (torch.bfloat16, eb.EGG_BF16) if dtype == "bf16" else (torch.float32, eb.EGG_F32)
    g = torch.Generator("cuda").manual_seed(d_in)
    W = (torch.randn((d_out, d_in), generator=g, device="cuda") * d_in ** -0.5).to(tdt)
    X = torch.randn((N * S, d_in), generator=g, device="cuda").to(tdt)
    Y = torch.full((N * S, d_out), float("nan"), dtype=tdt, device="cuda")
    key, sigma = eb.make_key(1, 2, 3), 0.5
    A, B = factors(ctx, key, N, d_out, rank, 0, tdt, code), factors(ctx, key, N, d_in, rank, 1, tdt, code)
    Ac, Bc = (torch.empty_like(A), torch.empty_like(B)) if cache else (None, None)
    ctx.eggroll_perturbed_forward(key, eb.make_shape(0, N, S, d_out, d_in, rank), sigma, eb.EGG_ACT_NONE, W, X, Y, Ac, Bc)
    if cache:
        assert torch.equal(A, Ac) and torch.equal(B, Bc)
    t = torch.bmm(X.double().view(N, S, d_in), B.double())
    corr = torch.bmm(t, A.double().transpose(1, 2).contiguous()).view(N * S, d_out) * (sigma / math.sqrt(rank))
    ref = X.double() @ W.double().t().contiguous() + corr
    rms = ref.square().mean(1, keepdim=True).sqrt()
    tol = 1e-5 * (ref.abs() + rms) if dtype == "f32" else 2.0 ** -8 * ref.abs() + 1e-4 * (rms + corr.abs().amax(1, keepdim=True))
    assert ((Y.double() - ref).abs() <= tol).all()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d_out,d_in,N,rank", [(4, 2, 1, 1), (36, 7, 9, 2), (260, 130, 33, 1), (256, 256, 257, 8), (1028, 1056, 64, 1),
                                              (1028, 1056, 65, 4), (2052, 1030, 40, 1),  # the 32 form, the 64 form, past both
                                              (3004, 2002, 40, 1), (3072, 2048, 33, 4)])  # 384 tiles of 128 x 128; in fp32 128 x 64
@pytest.mark.parametrize("w", [None, "bf16", "f32"])
def test_small_update(ctx, dtype, d_out, d_in, N, rank, w):
    import torch
    tdt, code = (torch.bfloat16, eb.EGG_BF16) if dtype == "bf16" else (torch.float32, eb.EGG_F32)
    g = torch.Generator("cuda").manual_seed(d_in)
    key = eb.make_key(1, 2, 3)
    A, B = factors(ctx, key, N, d_out, rank, 0, tdt, code), factors(ctx, key, N, d_in, rank, 1, tdt, code)
    f = torch.randn(N, generator=g, device="cuda")
    G0 = torch.randn((d_out, d_in), generator=g, device="cuda")
    G, W = G0.clone(), None
    if w:
        W0 = torch.randn((d_out, d_in), generator=g, device="cuda").to(torch.bfloat16 if w == "bf16" else torch.float32)
        W = W0.clone()
    ctx.eggroll_update(key, eb.make_shape(0, N, 1, d_out, d_in, rank), code, f, 0.25, 1, G, W, 0.125)
    ref = torch.einsum("nor,nir->oi", (A.double() * f.double()[:, None, None]).cpu(), B.double().cpu()).cuda() * 0.25 + G0.double()
    rms = ref.square().mean().sqrt()
    assert ((G.double() - ref).abs() <= (1e-5 * (ref.abs() + rms) if dtype == "f32" else 2e-3 * (ref.abs() + rms))).all()
    if w:
        want = W0.double() + 0.125 * G.double()
        assert ((W.double() - want).abs() <= (2.0 ** -8 if w == "bf16" else 1e-6) * (want.abs() + 1e-3)).all()


@pytest.mark.parametrize("d_out,d_in,S,rank,members", [
    (256, 264, 64, 1, (1, 8, 64, 700)), (256, 256, 64, 1, (1, 8, 64, 700)), (256, 128, 64, 4, (1, 8, 64, 600)), (256, 64, 128, 8, (1, 300)), (256, 328, 100, 4, (1, 8, 64, 500)), (512, 200, 16, 8, (3, 40, 300, 2500)), (256, 72, 31, 16, (2, 20, 200, 1600)),
    (384, 136, 1, 1, (2, 300, 4000, 30000)), (384, 136, 3, 4, (2, 100, 1300, 10000)), (256, 520, 14, 2, (2, 30, 300, 2500))])
@pytest.mark.parametrize("sigma,form", [(0.0, "plain"), (0.5, "plain"), (0.5, "gelu"), (0.5, "residual"), (0.5, "both")])
def test_bf16_rows_do_not_depend_on_the_call(ctx, d_out, d_in, S, rank, members, sigma, form):
    """A member's outputs are the same bits in a call of one member and in one of thousands: every kernel runs the same chain of
    MFMAs (16 x 16 blocks from memory, 128 x 128 tiles with two and four stages, 256 x 256 tiles, with
    the correction's operands from memory or parked)."""
    import torch
    N = max(members)
    g = torch.Generator("cuda").manual_seed(S)
    W = (torch.randn((d_out, d_in), generator=g, device="cuda") * d_in ** -0.5).to(torch.bfloat16)
    X = torch.randn((N * S, d_in), generator=g, device="cuda").to(torch.bfloat16)
    R = torch.randn((N * S, d_out), generator=g, device="cuda").to(torch.bfloat16)
    key = eb.make_key(1, 2, 3)

    def run(first, n):
        x, r = X[first * S:(first + n) * S].contiguous(), R[first * S:(first + n) * S].contiguous()
        y = torch.empty((n * S, d_out), dtype=torch.bfloat16, device="cuda")
        args = (key, eb.make_shape(first, n, S, d_out, d_in, rank), sigma, eb.EGG_ACT_GELU if form in ("gelu", "both") else eb.EGG_ACT_NONE, W, x)
        if form in ("residual", "both"):
            ctx.eggroll_perturbed_forward_add(*args, r, y)
        else:
            ctx.eggroll_perturbed_forward(*args, y)
        return y

    whole = run(0, N)
    for n in members[:-1]:
        for first in (0, N - n, (N - n) // 2):
            assert torch.equal(run(first, n), whole[first * S:(first + n) * S]), (first, n)


@pytest.mark.parametrize("d_out,d_in,N,S,rank,anti,cache", [
    (2044, 140, 1000, 1, 1, 0, 1), (2044, 140, 1000, 1, 1, 1, 0), (2044, 68, 333, 3, 4, 0, 0), (2044, 68, 500, 2, 1, 0, 1), (2044, 68, 333, 3, 8, 0, 0), (2044, 36, 60, 16, 16, 0, 1),   # 128 x 64 tiles
    (2044, 140, 2046, 1, 1, 1, 0), (2044, 140, 2047, 1, 1, 0, 1), (2044, 68, 681, 3, 2, 0, 0), (2044, 36, 60, 33, 8, 0, 0), (2044, 68, 510, 2, 16, 1, 0)])
@pytest.mark.parametrize("form", ["plain", "gelu", "residual", "both"])
def test_f32_tiles(ctx, d_out, d_in, N, S, rank, anti, cache, form):
    """fp32 layers of more than four 32 x 32 tiles per CU (128 x 64 tiles, then 128 x 128): factors regenerated in registers, shared by
    the lanes of a pair, or read; ragged in every direction.  GELU has a slope of at most 1.13."""
    import torch
    ids, per = N // (2 if anti else 1), S * (2 if anti else 1)
    g = torch.Generator("cuda").manual_seed(N)
    W = torch.randn((d_out, d_in), generator=g, device="cuda") * d_in ** -0.5
    X, R = (torch.randn((N * S, d), generator=g, device="cuda") for d in (d_in, d_out))
    Y = torch.full((N * S, d_out), float("nan"), device="cuda")
    key, sigma = eb.make_key(1, 2, 3), 0.5
    A, B = factors(ctx, key, ids, d_out, rank, 0, torch.float32, eb.EGG_F32), factors(ctx, key, ids, d_in, rank, 1, torch.float32, eb.EGG_F32)
    Ac, Bc = (torch.empty_like(A), torch.empty_like(B)) if cache else (None, None)
    args = (key, eb.make_shape(0, N, S, d_out, d_in, rank, anti), sigma, eb.EGG_ACT_GELU if form in ("gelu", "both") else eb.EGG_ACT_NONE, W, X)
    if form in ("residual", "both"):
        ctx.eggroll_perturbed_forward_add(*args, R, Y, Ac, Bc)
    else:
        ctx.eggroll_perturbed_forward(*args, Y, Ac, Bc)
    if cache:
        assert torch.equal(A, Ac) and torch.equal(B, Bc)
    t = torch.bmm(X.double().view(ids, per, d_in), B.double())
    if anti:
        t[:, S:] *= -1
    pre = X.double() @ W.double().t().contiguous() + torch.bmm(t, A.double().transpose(1, 2).contiguous()).view(N * S, d_out) * (sigma / math.sqrt(rank))
    ref = 0.5 * pre * (1 + torch.erf(pre * math.sqrt(0.5))) if form in ("gelu", "both") else pre
    ref = ref + R.double() if form in ("residual", "both") else ref
    assert ((Y.double() - ref).abs() <= 1e-5 * (ref.abs() + pre.square().mean(1, keepdim=True).sqrt())).all()


@pytest.mark.parametrize("S,rank,anti,members", [(1, 1, 0, (3, 500, 1000, 2048)), (1, 1, 1, (2, 500, 1000, 2048)), (1, 4, 0, (1, 300, 1001, 2000)),
                                                 (3, 2, 0, (1, 100, 333, 500)), (16, 16, 0, (1, 20, 61, 90))])
@pytest.mark.parametrize("sigma,form", [(0.0, "plain"), (0.5, "plain"), (0.5, "gelu"), (0.5, "residual"), (0.5, "both")])
def test_f32_rows_do_not_depend_on_the_call(ctx, S, rank, anti, members, sigma, form):
    """fp32 members are the same bits in any call, as the bf16 ones: 32 x 32 tiles (up to 1024 of them), 128 x 64 tiles, 128 x 128 tiles
    (the three larger member counts of each shape, in this order)."""
    import torch
    d_out, d_in, N = 2044, 140, max(members)
    g = torch.Generator("cuda").manual_seed(S)
    W = torch.randn((d_out, d_in), generator=g, device="cuda") * d_in ** -0.5
    X, R = (torch.randn((N * S, d), generator=g, device="cuda") for d in (d_in, d_out))
    key = eb.make_key(1, 2, 3)

    def run(first, n):
        x, r = X[first * S:(first + n) * S].contiguous(), R[first * S:(first + n) * S].contiguous()
        y = torch.empty((n * S, d_out), device="cuda")
        args = (key, eb.make_shape(first, n, S, d_out, d_in, rank, anti), sigma, eb.EGG_ACT_GELU if form in ("gelu", "both") else eb.EGG_ACT_NONE, W, x)
        if form in ("residual", "both"):
            ctx.eggroll_perturbed_forward_add(*args, r, y)
        else:
            ctx.eggroll_perturbed_forward(*args, y)
        return y

    whole = run(0, N)
    for n in members[:-1]:
        for first in (0, N - n, (N - n) // 4 * 2):
            assert torch.equal(run(first, n), whole[first * S:(first + n) * S]), (first, n)


@pytest.mark.parametrize("stages", range(1, 10))
@pytest.mark.parametrize("kind", ["f32", "bf16", "update"])
def test_counted_waits_equal_waits_for_everything(ctx, kind, stages):
    """The kernel that keeps four stages of K in flight waits for them by count; with the diagnostic switch it waits for every load.  The
    same bits, for row-major operands (32 x 32 tiles in fp32, 128 x 128 in bf16) and the update's K-packed panels, at every length of
    its loop's ends, whole and ragged last stages."""
    import torch
    for part in (0, 1):
        res = []
        for on in (0, 1):
            g = torch.Generator("cuda").manual_seed(stages)
            ctx.eggroll_set_conservative_waits(on)
            try:
                if kind == "update":
                    N = 64 * stages - 24 * part
                    f = torch.randn(N, generator=g, device="cuda")
                    Y = torch.empty((2048, 2040), device="cuda")   # 256 tiles of 128 x 128
                    ctx.eggroll_update(eb.make_key(1, 2, 3), eb.make_shape(0, N, 1, 2048, 2040, 1), eb.EGG_BF16, f, 1.0, 0, Y)
                else:
                    tdt, d_out, N, S = (torch.float32, 260, 30, 4) if kind == "f32" else (torch.bfloat16, 1028, 33, 16)
                    d_in = (32 if kind == "f32" else 64) * stages - 8 * part
                    W = torch.randn((d_out, d_in), generator=g, device="cuda").to(tdt)
                    X = torch.randn((N * S, d_in), generator=g, device="cuda").to(tdt)
                    Y = torch.empty((N * S, d_out), dtype=tdt, device="cuda")
                    ctx.eggroll_perturbed_forward(eb.make_key(1, 2, 3), eb.make_shape(0, N, S, d_out, d_in, 2), 0.5, eb.EGG_ACT_NONE, W, X, Y)
            finally:
                ctx.eggroll_set_conservative_waits(0)
            res.append(Y)
        assert torch.equal(res[0], res[1]) and torch.isfinite(res[0].float()).all()


@pytest.mark.parametrize("d_out,d_in,N,rank", [
    (2048, 1024, 1024, 1), (2048, 1024, 1025, 1), (1980, 1012, 515, 2),    # both sides of K = 1024 beside 16 tiles a row, ragged
    (512, 4096, 257, 4), (4096, 512, 1025, 1), (1472, 1344, 1025, 1), (1728, 1024, 1025, 1), (1792, 1024, 1025, 1),   # 64, 8 and 21 tiles a row; 432 tiles and 448
])
def test_bf16_update_of_deep_K(ctx, d_out, d_in, N, rank):
    """Tiles of 64 x 64 with K whole or split over the waves.  f a is rounded to fp16 once, 2^-11 of a term at most, uniformly: 2^-12 of the terms' norm with room to
    spare for the fp32 sums (1e-6); a single entry six times that."""
    import torch
    key, shape = eb.make_key(1, 2, 3), eb.make_shape(0, N, 1, d_out, d_in, rank)
    A, B = (torch.empty((N, d, rank), dtype=torch.bfloat16, device="cuda") for d in (d_out, d_in))
    ctx.eggroll_noise_gen(key, shape, eb.EGG_BF16, eb.EGG_NORMAL, 0, A, B)
    f = torch.randn(N, generator=torch.Generator("cuda").manual_seed(N), device="cuda")
    G, Gc = (torch.full((d_out, d_in), float("nan"), device="cuda") for _ in range(2))
    ctx.eggroll_update(key, shape, eb.EGG_BF16, f, 1.0, 0, G)
    ctx.eggroll_update(key, shape, eb.EGG_BF16, f, 1.0, 0, Gc, None, 0.0, A, B)
    assert torch.equal(G, Gc)
    a, b = (F.double().transpose(1, 2).reshape(N * rank, -1) for F in (A, B))
    a = a * f.double().repeat_interleave(rank)[:, None]
    ref, s = a.t().contiguous() @ b, (a.square().t().contiguous() @ b.square()).sqrt()
    err = (G.double() - ref).abs()
    assert err.norm() <= 2.0 ** -12 * s.norm() and (err <= 6 * 2.0 ** -12 * s).all()
