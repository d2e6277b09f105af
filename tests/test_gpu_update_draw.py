"""GPU: updates of small populations, whose factors are drawn in the kernel that multiplies them.

The same bits as from the same factors in the caller's caches, which are packed and multiplied by other kernels, for ragged tiles, K that ends
inside a step, a first member other than 0, both weight types, accumulation, and fitness that is all zero or holds an infinity."""
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


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("d_out,d_in,N,rank,kind", [
    (8, 8, 1, 1, "normal"), (32, 32, 3, 2, "normal"), (36, 68, 5, 16, "normal"), (100, 264, 33, 1, "zero"), (264, 100, 31, 4, "inf"),
    (64, 96, 128, 1, "normal"), (64, 96, 129, 1, "normal"), (64, 96, 65, 1, "normal"), (72, 64, 16, 8, "normal"), (256, 256, 64, 1, "normal"), (1024, 512, 32, 4, "normal"), (1024, 512, 16, 4, "normal"), (1028, 512, 64, 1, "normal"),
])
def test_the_bits_of_cached_factors(ctx, dtype, d_out, d_in, N, rank, kind):
    import torch
    tdt, code = (torch.bfloat16, eb.EGG_BF16) if dtype == "bf16" else (torch.float32, eb.EGG_F32)
    first, key = 17, eb.make_key(8, 9, 10)
    shape = eb.make_shape(first, N, 1, d_out, d_in, rank)
    g = torch.Generator("cuda").manual_seed(N)
    f = torch.randn(N, generator=g, device="cuda")
    if kind == "zero":
        f.zero_()
    if kind == "inf":
        f[N // 2] = float("inf")
    A, B = (torch.empty((N, d, rank), dtype=tdt, device="cuda") for d in (d_out, d_in))
    ctx.eggroll_noise_gen(key, shape, code, eb.EGG_NORMAL, 0, A, B)
    G0 = torch.randn((d_out, d_in), generator=g, device="cuda")
    for accumulate, w in ((0, None), (1, tdt), (0, torch.float32)):
        W0 = None if w is None else torch.randn((d_out, d_in), generator=g, device="cuda").to(w)
        got = []
        for caches in ((None, None), (A, B)):
            G = G0.clone() if accumulate else torch.full_like(G0, float("nan"))
            W = None if w is None else W0.clone()
            ctx.eggroll_update(key, shape, code, f, 0.5, accumulate, G, W, 0.125, *caches)
            got.append((G,) if w is None else (G, W))
        for x, y in zip(*got):
            assert torch.equal(x.isnan(), y.isnan()) and torch.equal(x[~x.isnan()], y[~x.isnan()])
            assert kind == "inf" or not x.isnan().any()
