"""GPU: few members with many rows, whose projections are formed by several workgroups each from factors drawn beforehand.

A member's outputs are the same bits as in a call with so many members that each has one workgroup, and as in the call that
allocates nothing (every workgroup draws the factors again); against 64 bits from the library's own factors as in the other layers: fp32 1e-5
of |value| + rms, bf16 one rounding, 2^-8."""
import math

import pytest

from helpers import memory_left
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


def test_little_memory():
    """Where there is no memory for the factors drawn beforehand every workgroup draws its member's: the same bits."""
    import torch
    d_out, d_in, N, S, rank = 32, 1 << 21, 16, 64, 16   # factors B of 1 GB
    g = torch.Generator("cuda").manual_seed(4)
    W, X = ((torch.randn((n, d_in), generator=g, device="cuda") * 1e-3).to(torch.bfloat16) for n in (d_out, N * S))

    def forward():
        Y = torch.empty((N * S, d_out), dtype=torch.bfloat16, device="cuda")
        c = eb.Context(0)
        try:
            c.eggroll_perturbed_forward(eb.make_key(1, 2, 3), eb.make_shape(0, N, S, d_out, d_in, rank), 0.5, eb.EGG_ACT_NONE, W, X, Y)
            torch.cuda.synchronize()
        finally:
            c.close()
        return Y

    want = forward()
    with memory_left(700 << 20):
        got = forward()
    assert torch.equal(got, want)


@pytest.mark.parametrize("call", ["forward", "update"])
def test_scratch_to_be_had_only_outside_a_capture(call):
    """Calls whose faster form wants scratch that no call before them needed run in a capture all the same, without it."""
    import torch
    d, rank, S = 1024, 4, 64
    few, many = (24, 800) if call == "forward" else (224, 240)   # (the larger call leaves scratch for all but the faster form)
    g = torch.Generator("cuda").manual_seed(4)
    stream = torch.cuda.Stream()
    ctx = eb.Context(0, stream=stream)
    key = eb.make_key(1, 2, 3)
    if call == "forward":
        W, X = ((torch.randn((n, d), generator=g, device="cuda")).to(torch.bfloat16) for n in (d, many * S))
        out = torch.zeros((many * S, d), dtype=torch.bfloat16, device="cuda")

        def run(c, n):
            c.eggroll_perturbed_forward(key, eb.make_shape(0, n, S, d, d, rank), 0.5, eb.EGG_ACT_NONE, W, X, out)
    else:
        f, out = torch.randn(many, generator=g, device="cuda"), torch.zeros((d, d), device="cuda")
        A, B = (torch.zeros((many, d, 1), device="cuda") for _ in range(2))

        def run(c, n, *caches):
            c.eggroll_update(key, eb.make_shape(0, n, 1, d, d, 1), eb.EGG_F32, f, 1.0, 0, out, None, 0.0, *caches)

    other = eb.Context(0, stream=stream)
    with torch.cuda.stream(stream):
        run(other, few)                             # (the reference; code is loaded outside the capture)
        want = out.clone()
        run(ctx, many, *((A, B) if call == "update" else ()))
    torch.cuda.synchronize()
    generation = ctx.eggroll_scratch_generation()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=stream):
        run(ctx, few)
    assert ctx.eggroll_scratch_generation() == generation
    for _ in range(3):
        out.zero_()
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        if call == "forward":
            assert torch.equal(out[:few * S], want[:few * S])
        else:
            assert (out - want).norm() <= 1e-6 * want.norm()   # (fp32 products for those of parts)
    ctx.close()
    other.close()
