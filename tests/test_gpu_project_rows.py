"""GPU: projections of rank 8 and 16 with two and four rows of a wave at once, at the edges of the rule between them and of a step.

t is seen through a layer with W = 0: Y = c t A^T, against the same in 64 bits from the library's own factors.  fp32 outputs: t is an
fp32 sum of up to 4104 products (random signs, 2^-24 sqrt(d_in) of the rms each way, 2e-6 at most), so 2e-5 of |row| covers it and the
rank-16 sum that follows."""
import math

import pytest

from paper_2511_16652_amd import binding as eb

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,S,d_in,rank,anti", [
    ("bf16", 7, 8, 8, 0), ("bf16", 8, 1016, 8, 0), ("bf16", 15, 1024, 8, 0), ("bf16", 16, 1032, 16, 0), ("bf16", 23, 4104, 8, 0), ("bf16", 64, 2056, 16, 0),
    ("bf16", 8, 520, 8, 1), ("f32", 8, 4, 8, 0), ("f32", 15, 508, 16, 0), ("f32", 16, 516, 8, 0), ("f32", 47, 1028, 8, 0), ("f32", 4, 1024, 16, 1),
    ("f32", 16, 4100, 16, 0),   # factors in several panels of LDS
])
def test_rows_at_once(dtype, S, d_in, rank, anti):
    import torch
    tdt, code = (torch.bfloat16, eb.EGG_BF16) if dtype == "bf16" else (torch.float32, eb.EGG_F32)
    N, d_out, sigma = 6, 64, 0.5
    ids = N // (2 if anti else 1)
    ctx = eb.Context(0)
    key = eb.make_key(5, 6, 7)
    A = torch.empty((ids, d_out, rank), dtype=tdt, device="cuda")
    B = torch.empty((ids, d_in, rank), dtype=tdt, device="cuda")
    ctx.eggroll_noise_gen(key, eb.make_shape(0, ids, 1, d_out, d_in, rank), code, eb.EGG_NORMAL, 0, A, B)
    X = torch.randn((N * S, d_in), generator=torch.Generator("cuda").manual_seed(S), device="cuda").to(tdt)
    W = torch.zeros((d_out, d_in), dtype=tdt, device="cuda")
    Y = torch.full((N * S, d_out), float("nan"), dtype=torch.float32, device="cuda")
    ctx.eggroll_perturbed_forward(key, eb.make_shape(0, N, S, d_out, d_in, rank, antithetic=bool(anti)), sigma, eb.EGG_ACT_NONE, W, X, Y)
    rows = N * S // ids
    t = torch.bmm(X.double().view(ids, rows, d_in), B.double())
    ref = torch.bmm(t, A.double().transpose(1, 2).contiguous()) * (sigma / math.sqrt(rank))
    if anti:
        ref[:, S:] *= -1
    ref = ref.view(N * S, d_out)
    err = (Y.double() - ref).norm(dim=1) / ref.norm(dim=1)
    assert err.max() <= 2e-5
    torch.cuda.synchronize()
    ctx.close()


@pytest.mark.parametrize("rank", [1, 2, 4, 8, 16])
@pytest.mark.parametrize("S", [2, 8, 16])
def test_the_order_over_lanes(rank, S):
    """A row's products are added over the 64 lanes as a butterfly does it: lanes 32 apart first, then 16, 8, 4, 2, 1 (fixed, so that a
    layer's bits stay what they were when the pass is changed).  One column per lane is not zero, so the order of a lane's own sum does
    not matter; c = 1 and W = 0, so Y is a chain of fused multiply-adds of t and A, emulated with 64 bits of mantissa.  Exact."""
    import numpy as np
    import torch
    N, d_in, d_out = 3, 256, 8
    ctx = eb.Context(0)
    key = eb.make_key(21, 22, 23)
    A, B = (torch.empty((N, d, rank), device="cuda") for d in (d_out, d_in))
    ctx.eggroll_noise_gen(key, eb.make_shape(0, N, 1, d_out, d_in, rank), eb.EGG_F32, eb.EGG_NORMAL, 0, A, B)
    X = torch.zeros((N * S, d_in), device="cuda")
    X[:, ::4] = torch.randn((N * S, 64), generator=torch.Generator("cuda").manual_seed(rank), device="cuda")
    W, Y = torch.zeros((d_out, d_in), device="cuda"), torch.empty((N * S, d_out), device="cuda")
    sigma = float(np.sqrt(np.float32(rank)))
    ctx.eggroll_perturbed_forward(key, eb.make_shape(0, N, S, d_out, d_in, rank), sigma, eb.EGG_ACT_NONE, W, X, Y)
    a, b, x = A.cpu().numpy(), B.cpu().numpy()[:, ::4], X.cpu().numpy().reshape(N, S, d_in)[:, :, ::4]
    t = x[:, :, :, None] * b[:, None]            # fp32 products [member][row][lane][rank]
    while t.shape[2] > 1:
        half = t.shape[2] // 2
        t = t[:, :, :half] + t[:, :, half:]
    want = np.zeros((N, S, d_out), np.float32)
    for l in range(rank):
        want = (t[:, :, 0, l, None].astype(np.longdouble) * a[:, None, :, l].astype(np.longdouble) + want).astype(np.float32)
    assert (Y.cpu().numpy().reshape(N, S, d_out) == want).all()
    torch.cuda.synchronize()
    ctx.close()
