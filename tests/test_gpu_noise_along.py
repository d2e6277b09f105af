"""GPU: the factors A of a layer, drawn in the launch of its projections by workgroups after the members'.

A is what the noise entry point draws, wherever it went with the projections or not (vectors that are not whole 16-byte pieces, more of it
than goes along beside a large panel), and the outputs are the same bits with and without the caller's caches; against 64 bits from the
library's own factors as in the other layers: fp32 1e-5 of |value| + rms, bf16 one rounding, 2^-8."""
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


@pytest.mark.parametrize("dtype,d_out,d_in,N,S,rank,anti", [
    ("bf16", 4, 64, 300, 2, 1, False),        # half a piece a member: a launch of its own
    ("bf16", 8, 72, 1, 2, 1, False), ("bf16", 12, 72, 301, 3, 2, False), ("bf16", 24, 64, 85, 1, 16, False), ("bf16", 100, 520, 6, 1, 2, True),
    ("bf16", 1028, 264, 513, 1, 4, False), ("bf16", 200, 264, 514, 5, 8, True), ("bf16", 64, 72, 2, 1, 1, True),
    ("bf16", 2048, 8712, 256, 2, 4, False), ("bf16", 2056, 8712, 256, 2, 4, False),  # the most, and more, beside 70 KB of LDS
    # pairs of one row at rank 1, whose A is read back from a cache and drawn again without one: both factors along, A apart, tiles of 32, 64, 128 and 256
    ("bf16", 100, 72, 300, 1, 1, True), ("bf16", 1032, 264, 600, 1, 1, True), ("bf16", 2056, 520, 1100, 1, 1, True), ("bf16", 4104, 264, 4200, 1, 1, True),
    ("f32", 72, 68, 300, 1, 1, True), ("f32", 1028, 260, 1100, 1, 1, True), ("f32", 2052, 260, 2100, 1, 1, True),
    # few members with many rows and A of half pieces: each of several workgroups draws its member's B, the first fills the cache
    ("bf16", 380, 16, 6, 16, 1, False), ("bf16", 100, 24, 2, 17, 1, False), ("bf16", 20, 4104, 4, 40, 1, True), ("bf16", 4, 66000, 3, 70, 1, False),
    ("f32", 2048, 1024, 640, 2, 16, False), ("f32", 2052, 1024, 640, 2, 16, False),   # the same beside 64 KB, in fp32
    ("f32", 4, 64, 300, 2, 1, False), ("f32", 36, 68, 258, 1, 2, True), ("f32", 260, 2052, 515, 3, 16, False), ("f32", 132, 128, 600, 4, 4, True),
])
def test_the_factors_are_the_entry_points(ctx, dtype, d_out, d_in, N, S, rank, anti):
    import torch
    tdt, code = (torch.bfloat16, eb.EGG_BF16) if dtype == "bf16" else (torch.float32, eb.EGG_F32)
    sigma, key, first = 0.5, eb.make_key(5, 6, 7), 10
    g = torch.Generator("cuda").manual_seed(d_in + N)
    W = (torch.randn((d_out, d_in), generator=g, device="cuda") * d_in ** -0.5).to(tdt)
    X = torch.randn((N * S, d_in), generator=g, device="cuda").to(tdt)
    shape = eb.make_shape(first, N, S, d_out, d_in, rank, anti)

    def forward(call, *caches):
        y = torch.full((N * S, d_out), float("nan"), dtype=tdt, device="cuda")
        call(key, shape, sigma, eb.EGG_ACT_NONE, W, X, y, *caches)
        return y

    ids = N // 2 if anti else N
    A, B, A2, B2 = (torch.full((ids, d, rank), float("nan"), dtype=tdt, device="cuda") for d in (d_out, d_in, d_out, d_in))
    Y = forward(ctx.eggroll_perturbed_forward, A, B)
    assert torch.equal(Y, forward(ctx.eggroll_perturbed_forward, None, None))
    assert torch.equal(Y, forward(ctx.eggroll_perturbed_forward_noalloc, A2, None))
    assert torch.equal(A, A2)
    ctx.eggroll_noise_gen(key, eb.make_shape(first // 2 if anti else first, ids, 1, d_out, d_in, rank), code, eb.EGG_NORMAL, 0, A2, B2)
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
