"""GPU: the bf16 layer whose correction is folded into the accumulators for row groups of any length, at the edges of its
dispatch: both sides of the smallest row group (15 rows of one noise id; a pair counts its 2S rows), blocks that straddle two
members, rank 16's second pass, ragged K, d_out and row counts, both tile sizes.

Reference in 64 bits from the factors that eggroll_noise_gen writes.  Per entry: one bf16 rounding (2^-9 of the value), the
fp32 sums and the hi/lo split of c t (2^-16 of the correction, of the size of the row) and the polynomial GELU (1.3e-4)."""
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


CASES = [  # d_out, d_in, members, S, rank, antithetic, gelu, residual
    (132, 72, 9, 15, 1, 0, 0, 0),
    (132, 72, 9, 14, 1, 0, 0, 0),      # below the rule: the general epilogue
    (260, 136, 7, 16, 2, 0, 1, 0),
    (124, 200, 6, 17, 4, 0, 0, 1),
    (388, 64, 5, 31, 8, 0, 1, 1),
    (136, 72, 9, 15, 16, 0, 0, 0),
    (136, 72, 4, 100, 16, 0, 0, 1),
    (200, 264, 8, 8, 2, 1, 0, 0),      # pairs: 16 rows share their factors
    (200, 264, 8, 7, 2, 1, 0, 0),      # 14: the general epilogue
    (64, 8, 1, 1, 1, 0, 0, 0),
    (4096, 72, 31, 100, 4, 0, 1, 0),   # 256 x 256 tiles, ragged K
    (4100, 128, 195, 17, 8, 0, 0, 1),
    (4096, 64, 205, 15, 16, 0, 0, 0),
    (4096, 128, 62, 51, 1, 0, 0, 0),
    (4096, 72, 50, 64, 2, 0, 0, 0),    # S a multiple of 64, ragged K
    (2052, 72, 26, 100, 4, 0, 1, 0),   # 257 to 512 tiles of 128 x 128, two workgroups per CU: ragged K, blocks of two members
    (2052, 136, 51, 51, 16, 0, 0, 1),
    (2052, 200, 100, 26, 2, 0, 1, 1),
    (2052, 64, 41, 64, 1, 0, 0, 1),
    (2052, 72, 52, 50, 8, 1, 0, 0),
]


@pytest.mark.parametrize("case", CASES)
@pytest.mark.parametrize("sigma", [0.0, 0.7])
def test_folded_layer(ctx, case, sigma):
    import torch
    d_out, d_in, N, S, rank, anti, gelu, resid = case
    R, ids, per = N * S, N // (2 if anti else 1), S * (2 if anti else 1)
    g = torch.Generator("cuda").manual_seed(d_out + S)
    draw = lambda *s: torch.randn(s, generator=g, device="cuda").to(torch.bfloat16)  # noqa: E731
    W, X, Rin = draw(d_out, d_in) * d_in ** -0.5, draw(R, d_in), draw(R, d_out)
    Y = torch.full((R, d_out), float("nan"), dtype=torch.bfloat16, device="cuda")
    key, shape = eb.make_key(3, 2, 5), eb.make_shape(4, N, S, d_out, d_in, rank, anti)
    act = eb.EGG_ACT_GELU if gelu else eb.EGG_ACT_NONE
    if resid:
        ctx.eggroll_perturbed_forward_add(key, shape, sigma, act, W, X, Rin, Y)
    else:
        ctx.eggroll_perturbed_forward(key, shape, sigma, act, W, X, Y)
    A = torch.empty((ids, d_out, rank), dtype=torch.bfloat16, device="cuda")
    B = torch.empty((ids, d_in, rank), dtype=torch.bfloat16, device="cuda")
    ctx.eggroll_noise_gen(key, eb.make_shape(4 // (2 if anti else 1), ids, 1, d_out, d_in, rank), eb.EGG_BF16, eb.EGG_NORMAL, 0, A, B)
    t = torch.bmm(X.double().view(ids, per, d_in), B.double())
    if anti:
        t[:, S:] *= -1
    corr = torch.bmm(t, A.double().transpose(1, 2).contiguous()).view(R, d_out) * (sigma / math.sqrt(rank))
    pre = X.double() @ W.double().t().contiguous() + corr
    ref = 0.5 * pre * (1 + torch.erf(pre * math.sqrt(0.5))) if gelu else pre
    if resid:
        ref = ref + Rin.double()
    tol = 2.0 ** -8 * ref.abs() + 1e-4 * (1 + corr.abs().amax(1, keepdim=True)) + (2e-4 if gelu else 0)
    err = (Y.double() - ref).abs()
    assert torch.isfinite(Y.float()).all() and (err <= tol).all(), (err - tol).max()


@pytest.mark.parametrize("shape", [(132, 72, 9, 17), (1028, 72, 30, 17), (2052, 72, 26, 100), (4096, 64, 62, 51), (4096, 72, 62, 51)])
@pytest.mark.parametrize("rank", [1, 4, 8])
@pytest.mark.parametrize("gelu,resid", [(0, 0), (1, 0), (0, 1), (1, 1)])
def test_every_form(ctx, shape, rank, gelu, resid):
    """Each width of the lanes' factors with each activation and residual, in each of the folding kernels."""
    d_out, d_in, N, S = shape
    for sigma in (0.0, 0.7) if rank == 1 else (0.7,):
        test_folded_layer(ctx, (d_out, d_in, N, S, rank, 0, gelu, resid), sigma)


@pytest.mark.parametrize("d_out,d_in,N,S", [(64, 64, 3, 15), (64, 64, 2, 100), (260, 72, 9, 31), (1028, 64, 37, 16), (4096, 64, 130, 64), (4096, 72, 84, 100)])
@pytest.mark.parametrize("rank", [1, 2, 4, 8, 16])
def test_an_infinite_projection(ctx, d_out, d_in, N, S, rank):
    """Two rows whose projections overflow (their products with W do not: the columns are zero there): their outputs are infinite with the
    sign of the correction, NaN only where infinities of both signs meet; the other rows, of the same blocks too, are untouched."""
    import torch
    R, sigma = N * S, 1e-30  # a projection that stays finite contributes next to nothing
    g = torch.Generator("cuda").manual_seed(rank)
    W = (torch.randn((d_out, d_in), generator=g, device="cuda") * d_in ** -0.5).to(torch.bfloat16)
    X = torch.randn((R, d_in), generator=g, device="cuda").to(torch.bfloat16)
    W[:, :32] = 0
    rows = [S + 1, R - 2]
    key = eb.make_key(3, 2, 5)
    A = torch.empty((N, d_out, rank), dtype=torch.bfloat16, device="cuda")
    B = torch.empty((N, d_in, rank), dtype=torch.bfloat16, device="cuda")
    ctx.eggroll_noise_gen(key, eb.make_shape(0, N, 1, d_out, d_in, rank), eb.EGG_BF16, eb.EGG_NORMAL, 0, A, B)
    for q in rows:
        b = B[q // S, :32].abs().float().sort(-1).values
        at = int((b[:, -1] - (b[:, -2] if rank > 1 else 0)).argmax())  # one rank term stands out: it alone overflows
        X[q, at] = 3.5e38 / b[at, -1].double()
    Y = torch.empty((R, d_out), dtype=torch.bfloat16, device="cuda")
    ctx.eggroll_perturbed_forward(key, eb.make_shape(0, N, S, d_out, d_in, rank), sigma, eb.EGG_ACT_NONE, W, X, Y)
    plain = X.double() @ W.double().t().contiguous()
    seen = 0
    for q in rows:
        t = (X[q].double()[:, None] * B[q // S].double()).sum(0)
        t = torch.where(t.abs() >= 2.0 ** 128 - 2.0 ** 103, t.sign() * math.inf, t * (sigma / math.sqrt(rank)))  # as fp32 holds it
        want = plain[q] + (A[q // S].double() * t).sum(-1)
        seen += int(torch.isinf(want).sum())
        assert torch.equal(torch.isnan(Y[q]), torch.isnan(want)) and torch.equal(torch.isposinf(Y[q]), torch.isposinf(want)) and torch.equal(
            torch.isneginf(Y[q]), torch.isneginf(want))
    assert seen
    rest = torch.ones(R, dtype=torch.bool)
    rest[rows] = False
    assert ((Y.double() - plain).abs() <= 2.0 ** -8 * plain.abs() + 1e-5)[rest].all()


@pytest.mark.parametrize("S", [15, 64, 100])
def test_a_projection_beyond_bf16(ctx, S):
    """c t between the largest bf16 value and the largest fp32 value (W = 0, rank 1): Y = c t A, not infinity."""
    import torch
    d_out, d_in, N, key = 260, 64, 4, eb.make_key(3, 2, 6)
    A = torch.empty((N, d_out, 1), dtype=torch.bfloat16, device="cuda")
    B = torch.empty((N, d_in, 1), dtype=torch.bfloat16, device="cuda")
    ctx.eggroll_noise_gen(key, eb.make_shape(0, N, 1, d_out, d_in, 1), eb.EGG_BF16, eb.EGG_NORMAL, 0, A, B)
    W, X = torch.zeros((d_out, d_in), dtype=torch.bfloat16, device="cuda"), torch.zeros((N * S, d_in), dtype=torch.bfloat16, device="cuda")
    b, q, target = B[1].double().view(-1), S + 3, 3.399e38
    at = int(b.abs().argmax())
    X[q, at] = (target / b[at]).to(torch.bfloat16)
    near = int((b.abs() - 0.5).abs().argmin())  # what is left of the target, to 2^-9 of 2^-9
    X[q, near] = ((target - X[q, at].double() * b[at]) / b[near]).to(torch.bfloat16)
    t = float((X[q].double() * b).sum())
    assert 3.3953e38 < t < 3.4028e38
    Y = torch.empty((N * S, d_out), dtype=torch.bfloat16, device="cuda")
    ctx.eggroll_perturbed_forward(key, eb.make_shape(0, N, S, d_out, d_in, 1), 1.0, eb.EGG_ACT_NONE, W, X, Y)
    want = t * A[1].double().view(-1)
    small = want.abs() < 3.3e38
    assert small.any() and ((Y[q].double() - want).abs() <= 2.0 ** -8 * want.abs())[small].all()
