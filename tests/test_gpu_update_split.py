"""GPU: fp32 updates whose generated factors are two fp16 parts each (more than 512 tiles of 32 x 32 on 256 CUs, 192 kappa and more), at the edges
of tiles, stages and the rule, against 64 bits from the library's own factors.

Bound: the rounding of products and parts, below 2^-23 of a term each, and of K / 32 partial sums: 2e-6 of the row and column norms'
product covers K up to 8192 (the largest error seen is below a third of it); what the rule leaves to fp32 is held to the same."""
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


def factors(ctx, key, begin, N, d_out, d_in, rank):
    import torch
    A, B = (torch.empty((N, d, rank), device="cuda") for d in (d_out, d_in))
    ctx.eggroll_noise_gen(key, eb.make_shape(begin, N, 1, d_out, d_in, rank), eb.EGG_F32, eb.EGG_NORMAL, 0, A, B)
    flat = lambda F: F.double().transpose(1, 2).reshape(N * rank, -1)  # noqa: E731
    return flat(A), flat(B)


@pytest.mark.parametrize("d_out,d_in,N,rank", [
    (1024, 736, 191, 1), (1024, 736, 192, 1), (1024, 512, 300, 1), (1024, 520, 193, 1),     # both sides of 192 kappa and of 512 tiles
    (1032, 1022, 97, 2), (736, 1029, 50, 4), (1000, 1000, 31, 8), (1028, 741, 13, 16),       # ragged; odd widths from rank 2 on
    (2048, 1028, 200, 1), (2052, 1026, 200, 1), (1400, 2100, 1025, 1), (4100, 300, 8192, 1),  # 64 | 128 tiles; the norm found beforehand
])
@pytest.mark.parametrize("w", [None, "bf16", "f32"])
def test_split_update(ctx, d_out, d_in, N, rank, w):
    import torch
    key, begin = eb.make_key(3, 1, 9), 5
    g = torch.Generator("cuda").manual_seed(N)
    f = torch.randn(N, generator=g, device="cuda") * 1e-20    # (any magnitude: a power of two is taken out)
    f[: N // 2] *= 1e-6
    G0 = torch.randn((d_out, d_in), generator=g, device="cuda")
    G = G0.clone()
    W0 = None if w is None else torch.randn((d_out, d_in), generator=g, device="cuda").to(torch.bfloat16 if w == "bf16" else torch.float32)
    W = None if w is None else W0.clone()
    scale, acc = 1e20, 1 if w == "f32" else 0
    args = (key, eb.make_shape(begin, N, 1, d_out, d_in, rank), eb.EGG_F32, f, scale, acc, G) + (() if w is None else (W, 0.125))
    ctx.eggroll_update(*args)
    A, B = factors(ctx, key, begin, N, d_out, d_in, rank)
    A *= f.double().repeat_interleave(rank)[:, None]
    ref = scale * (A.t().contiguous() @ B)
    tol = 2e-6 * scale * A.norm(dim=0)[:, None] * B.norm(dim=0)[None, :] / (N * rank) ** 0.5 * 3
    if acc:
        ref, tol = ref + G0.double(), tol + 2.0 ** -23 * (ref.abs() + G0.double().abs())
    assert ((G.double() - ref).abs() <= tol).all()
    if w:
        want = W0.double() + 0.125 * G.double()
        assert ((W.double() - want).abs() <= (2.0 ** -8 if w == "bf16" else 2.0 ** -22) * (want.abs() + 1e-3)).all()


@pytest.mark.parametrize("bad", [float("inf"), float("-inf"), float("nan"), "both", "large"])
def test_fitness_that_is_not_finite(ctx, bad):
    """An infinite fitness gives the infinities of its products, a NaN one NaN, whatever stands beside it."""
    import torch
    d_out, d_in, N, key = 1024, 736, 200, eb.make_key(3, 1, 9)
    f = torch.randn(N, generator=torch.Generator("cuda").manual_seed(1), device="cuda")
    if bad == "both":
        f[7], f[150] = float("inf"), float("-inf")
    elif bad == "large":
        f[7], f[9] = float("inf"), 3e37   # (its entries stay finite in fp32)
    else:
        f[7] = bad
    G = torch.zeros((d_out, d_in), device="cuda")
    ctx.eggroll_update(key, eb.make_shape(0, N, 1, d_out, d_in, 1), eb.EGG_F32, f, 1.0, 0, G)
    A, B = factors(ctx, key, 0, N, d_out, d_in, 1)
    k = [i for i in range(N) if not torch.isfinite(f[i])]
    ref = sum((f[i].double() * A[i])[:, None] * B[i][None, :] for i in k)   # the terms that decide the class
    assert torch.equal(torch.isnan(G), torch.isnan(ref)) and torch.equal(torch.isposinf(G), torch.isposinf(ref)) and torch.equal(torch.isneginf(G), torch.isneginf(ref))
