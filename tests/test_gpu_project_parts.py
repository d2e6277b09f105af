"""GPU: few members with many rows, whose projections are formed by several workgroups each from factors drawn beforehand.

A member's outputs are the same bits as in a call with so many members that each has one workgroup, and as in the call that
allocates nothing (every workgroup draws the factors again); against 64 bits from the library's own factors as in the other layers: fp32 1e-5
of |value| + rms, bf16 one rounding, 2^-8."""
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


@pytest.mark.parametrize("dtype,d_in,N,S,rank,anti", [
    ("bf16", 72, 1, 9, 1, False), ("bf16", 400, 2, 178, 8, False), ("bf16", 520, 3, 21, 2, False), ("bf16", 1032, 6, 79, 4, True),
    ("bf16", 8200, 2, 65, 1, True), ("bf16", 4104, 2, 37, 16, False), ("bf16", 4096, 2, 70, 4, False), ("bf16", 8192, 1, 100, 16, False),
    ("bf16", 264, 140, 40, 1, False), ("bf16", 1024, 256, 64, 1, False),   # the two limits of the number of members
    ("f32", 68, 1, 9, 1, False), ("f32", 1028, 3, 50, 2, False), ("f32", 2052, 2, 33, 16, True), ("f32", 300, 2, 130, 8, False), ("f32", 260, 3, 45, 4, False),
])
def test_parts_are_the_same_bits(ctx, dtype, d_in, N, S, rank, anti):
    import torch
    tdt, code = (torch.bfloat16, eb.EGG_BF16) if dtype == "bf16" else (torch.float32, eb.EGG_F32)
    d_out, sigma, key = 72, 0.5, eb.make_key(1, 2, 3)
    many = 1030 if anti else 515                     # more than two to a CU: one workgroup for each
    g = torch.Generator("cuda").manual_seed(d_in)
    W = (torch.randn((d_out, d_in), generator=g, device="cuda") * d_in ** -0.5).to(tdt)
    X = torch.randn((N * S, d_in), generator=g, device="cuda").to(tdt)
    Xm = torch.zeros((many * S, d_in), dtype=tdt, device="cuda")
    Xm[:N * S] = X

    def forward(call, x, n, caches):
        y = torch.full((n * S, d_out), float("nan"), dtype=tdt, device="cuda")
        call(key, eb.make_shape(0, n, S, d_out, d_in, rank, anti), sigma, eb.EGG_ACT_NONE, W, x, y, *caches)
        return y

    ids = N // 2 if anti else N
    A, B, A2, B2 = (torch.full((ids, d, rank), float("nan"), dtype=tdt, device="cuda") for d in (d_out, d_in, d_out, d_in))
    Y = forward(ctx.eggroll_perturbed_forward, X, N, (None, None))
    assert torch.equal(Y, forward(ctx.eggroll_perturbed_forward, X, N, (A, B)))
    assert torch.equal(Y, forward(ctx.eggroll_perturbed_forward, Xm, many, (None, None))[:N * S])
    assert torch.equal(Y, forward(ctx.eggroll_perturbed_forward_noalloc, X, N, (A2, None)))
    assert torch.equal(A, A2)
    ctx.eggroll_noise_gen(key, eb.make_shape(0, ids, 1, d_out, d_in, rank), code, eb.EGG_NORMAL, 0, A2, B2)
    assert torch.equal(A, A2) and torch.equal(B, B2)
    per = S * (2 if anti else 1)
    t = torch.bmm(X.double().view(ids, per, d_in), B.double())
    if anti:
        t[:, S:] *= -1
    corr = torch.bmm(t, A.double().transpose(1, 2).contiguous()).view(N * S, d_out) * (sigma / math.sqrt(rank))
    ref = X.double() @ W.double().t().contiguous() + corr
    rms = ref.square().mean(1, keepdim=True).sqrt()
    tol = 1e-5 * (ref.abs() + rms) if dtype == "f32" else 2.0 ** -8 * ref.abs() + 1e-4 * (rms + corr.abs().amax(1, keepdim=True))
    assert ((Y.double() - ref).abs() <= tol).all()
