"""GPU: bf16 layers of few tiles, in 32 x 32 and 64 x 64 tiles with four stages of K in flight, on both sides of each line of the rule between
them (on 256 CUs), with ragged K, rows and outputs.

A call's rows are the same bits as in a call of sixteen times the members, which runs in tiles of 128 and more; and one rounding from 64 bits, 2^-8 (plus what GELU's polynomial and the folded correction leave, 1e-4 of
the row's rms)."""
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


@pytest.mark.parametrize("d_out,d_in,N,S,rank,anti", [
    (512, 72, 32, 16, 2, 0),        # 16 x 16 tiles of 32
    (2048, 200, 16, 16, 1, 0), (2048, 200, 17, 16, 4, 0),      # 512 tiles of 32 | 544: 64 x 5 of 64
    (1028, 136, 30, 30, 16, 0),     # 17 x 15 of 64, ragged
    (1000, 520, 10, 100, 8, 0),     # 16 x 16 of 64
    (332, 264, 22, 128, 1, 1),      # 11 x 88 of 32, more than 256 of 64
    (2044, 392, 11, 91, 2, 0),      # 32 x 16 of 64, the most
    (516, 136, 600, 1, 1, 0), (1024, 136, 486, 1, 1, 0), (1020, 200, 1000, 1, 2, 0), (2048, 72, 1000, 1, 1, 1), (1284, 328, 300, 3, 4, 0), (1284, 64, 100, 9, 16, 0),
])
@pytest.mark.parametrize("form", ["plain", "gelu", "both"])
def test_few_tiles(ctx, d_out, d_in, N, S, rank, anti, form):
    import torch
    g = torch.Generator("cuda").manual_seed(d_in)
    bf = torch.bfloat16
    many, sigma, key = 16 * N, 0.5, eb.make_key(1, 2, 3)
    assert -(-d_out // 64) * -(-many * S // 64) > 512
    W = (torch.randn((d_out, d_in), generator=g, device="cuda") * d_in ** -0.5).to(bf)
    X, R = (torch.randn((many * S, d), generator=g, device="cuda").to(bf) for d in (d_in, d_out))

    def run(n):
        y = torch.full((n * S, d_out), float("nan"), dtype=bf, device="cuda")
        args = (key, eb.make_shape(0, n, S, d_out, d_in, rank, anti), sigma, eb.EGG_ACT_NONE if form == "plain" else eb.EGG_ACT_GELU, W, X[:n * S].contiguous())
        if form == "both":
            ctx.eggroll_perturbed_forward_add(*args, R[:n * S].contiguous(), y)
        else:
            ctx.eggroll_perturbed_forward(*args, y)
        return y

    Y = run(N)
    assert torch.equal(Y, run(many)[:N * S])
    ids, per = (N // 2, 2 * S) if anti else (N, S)
    A, B = (torch.empty((ids, d, rank), dtype=bf, device="cuda") for d in (d_out, d_in))
    ctx.eggroll_noise_gen(key, eb.make_shape(0, ids, 1, d_out, d_in, rank), eb.EGG_BF16, eb.EGG_NORMAL, 0, A, B)
    x = X[:N * S].double()
    t = torch.bmm(x.view(ids, per, d_in), B.double())
    if anti:
        t[:, S:] *= -1
    pre = x @ W.double().t().contiguous() + torch.bmm(t, A.double().transpose(1, 2).contiguous()).view(N * S, d_out) * (sigma / math.sqrt(rank))
    ref = pre if form == "plain" else 0.5 * pre * (1 + torch.erf(pre * math.sqrt(0.5)))
    ref = ref + R[:N * S].double() if form == "both" else ref
    assert ((Y.double() - ref).abs() <= 2.0 ** -8 * ref.abs() + 1e-4 * (1 + pre.square().mean(1, keepdim=True).sqrt())).all()


@pytest.mark.parametrize("sigma", [0.0, 0.5])
def test_rows_of_more_than_32_bits_of_offset(ctx, sigma):
    """A layer of a few outputs takes rows of any length: the last of these begins 4.4 GB behind the first."""
    import torch
    d_out, d_in, N = 32, (1 << 26) + (1 << 22) + 8, 2
    bf, key = torch.bfloat16, eb.make_key(1, 2, 3)
    g = torch.Generator("cuda").manual_seed(8)
    W, X = (torch.randn((n, d_in), generator=g, device="cuda", dtype=bf) for n in (d_out, N))
    Y = torch.full((N, d_out), float("nan"), dtype=bf, device="cuda")
    assert (d_out - 1) * d_in * 2 > 1 << 32
    ctx.eggroll_perturbed_forward(key, eb.make_shape(0, N, 1, d_out, d_in, 1), sigma, eb.EGG_ACT_NONE, W, X, Y)
    A, B = (torch.empty((N, d, 1), dtype=bf, device="cuda") for d in (d_out, d_in))
    ctx.eggroll_noise_gen(key, eb.make_shape(0, N, 1, d_out, d_in, 1), eb.EGG_BF16, eb.EGG_NORMAL, 0, A, B)
    ref, t, step = torch.zeros((N, d_out), dtype=torch.float64, device="cuda"), torch.zeros((N, 1), dtype=torch.float64, device="cuda"), 1 << 22
    for k in range(0, d_in, step):
        x = X[:, k:k + step].double()
        ref += x @ W[:, k:k + step].double().t().contiguous()
        t += (x * B[:, k:k + step, 0].double()).sum(1, keepdim=True)
    ref += sigma * t * A[:, :, 0].double()
    # one rounding, and an fp32 sum of 2^21 steps that rounds at the size of the whole: 2^-24 sqrt(2^21) of its deviation, ten times
    assert ((Y.double() - ref).abs() <= 2.0 ** -8 * ref.abs() + 1e-3 * d_in ** 0.5 * (1 + sigma)).all()
