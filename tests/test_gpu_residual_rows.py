"""GPU: the residual read ahead by the general forward epilogue (ragged tiles, few rows per member), in place and into another buffer, and
the factors of narrow projections, one block a thread.

Oracle: the same layer without the residual, fp32 output, from the same call; a bf16 output is that plus the residual, rounded once
more where the activation's bf16 grade allows it: 2^-8 of the sum and of each part.  In place and out of place: the same bits."""
import pytest

from paper_2511_16652_amd import binding as eb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d_out,d_in,N,S,rank,anti", [
    (1028, 512, 1100, 1, 1, 1), (1028, 264, 1101, 1, 1, 0),      # 128 x 128 tiles, factors in registers
    (1156, 256, 370, 3, 2, 0), (1028, 512, 222, 5, 4, 0),        # factors from memory
    (260, 136, 40, 3, 8, 0), (132, 72, 10, 2, 1, 1),              # small tiles; the residual at the store (rank 8)
    (3076, 64, 4100, 1, 1, 0), (4100, 64, 2050, 1, 2, 1),        # 256 x 256 and 256 x 128 tiles
])
def test_residual(d_out, d_in, N, S, rank, anti):
    import torch
    ctx = eb.Context(0)
    key, sigma = eb.make_key(8, 9, 10), 0.25
    g = torch.Generator("cuda").manual_seed(d_out)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda").to(torch.bfloat16)  # noqa: E731
    W, X, Rn = rnd(d_out, d_in) * d_in ** -0.5, rnd(N * S, d_in), rnd(N * S, d_out)
    shape = eb.make_shape(0, N, S, d_out, d_in, rank, anti)
    plain = torch.empty((N * S, d_out), device="cuda")
    ctx.eggroll_perturbed_forward(key, shape, sigma, eb.EGG_ACT_NONE, W, X, plain)
    Y = torch.full((N * S, d_out), float("nan"), dtype=torch.bfloat16, device="cuda")
    ctx.eggroll_perturbed_forward_add(key, shape, sigma, eb.EGG_ACT_NONE, W, X, Rn, Y)
    Z = Rn.clone()
    ctx.eggroll_perturbed_forward_add(key, shape, sigma, eb.EGG_ACT_NONE, W, X, Z, Z)
    assert torch.equal(Y, Z)
    ref = plain.double() + Rn.double()
    assert ((Y.double() - ref).abs() <= 2.0 ** -8 * (ref.abs() + plain.double().abs() + Rn.double().abs())).all()
    torch.cuda.synchronize()
    ctx.close()


@pytest.mark.parametrize("dtype,d_in,S,rank", [("bf16", 8, 2, 1), ("bf16", 1024, 3, 1), ("bf16", 1032, 3, 1), ("bf16", 512, 4, 4), ("bf16", 520, 4, 4), ("bf16", 128, 2, 16),
                                               ("f32", 4, 2, 1), ("f32", 512, 2, 1), ("f32", 516, 2, 1), ("f32", 32, 2, 16)])
def test_narrow_projection(dtype, d_in, S, rank):
    import torch
    tdt, code = (torch.bfloat16, eb.EGG_BF16) if dtype == "bf16" else (torch.float32, eb.EGG_F32)
    N, d_out = 7, 8
    ctx = eb.Context(0)
    key = eb.make_key(11, 12, 13)
    A, B = (torch.empty((N, d, rank), dtype=tdt, device="cuda") for d in (d_out, d_in))
    ctx.eggroll_noise_gen(key, eb.make_shape(0, N, 1, d_out, d_in, rank), code, eb.EGG_NORMAL, 0, A, B)
    Ac, Bc = torch.empty_like(A), torch.empty_like(B)
    X = torch.randn((N * S, d_in), generator=torch.Generator("cuda").manual_seed(d_in), device="cuda").to(tdt)
    W = torch.zeros((d_out, d_in), dtype=tdt, device="cuda")
    Y = torch.empty((N * S, d_out), device="cuda")
    ctx.eggroll_perturbed_forward(key, eb.make_shape(0, N, S, d_out, d_in, rank), 1.0, eb.EGG_ACT_NONE, W, X, Y, Ac, Bc)
    assert torch.equal(B, Bc) and torch.equal(A, Ac)
    Xm, Bm, Am = X.double().view(N, S, d_in), B.double(), A.double().transpose(1, 2).contiguous()
    ref = torch.bmm(torch.bmm(Xm, Bm), Am) * rank ** -0.5
    # a fp32 sum of n terms is off by at most n 2^-24 of the sum of their magnitudes: up to 32 additions in a lane, 6 across lanes, then
    # the rank's
    bound = torch.bmm(torch.bmm(Xm.abs(), Bm.abs()), Am.abs()) * rank ** -0.5 * (64 * 2.0 ** -24)
    assert ((Y.double().view(N, S, d_out) - ref).abs() <= bound).all()
    torch.cuda.synchronize()
    ctx.close()
