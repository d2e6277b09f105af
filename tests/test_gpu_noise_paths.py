"""GPU: the factor generators that work by 16-byte pieces or straight into the update's panels, at the edges of their ranges.

The pieces are held to the general kernel (one Threefry block a thread, taken for vectors that are not whole pieces) through
the stream's addressing: a vector of n values is the beginning of a longer one.  The generated panels are held to the packed
ones: the update from caches and the update that regenerates are the same bits.
"""
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


@pytest.mark.parametrize("dist", ["bf16", "f32", "raw", "int", "table"])
@pytest.mark.parametrize("members,n", [(1, 16), (3, 48), (257, 16), (100, 80), (5, 8208), (33, 1024)])
def test_pieces_equal_single_blocks(ctx, dist, members, n):
    import torch
    tdt, code, kind, bound = {"bf16": (torch.bfloat16, eb.EGG_BF16, eb.EGG_NORMAL, 0), "f32": (torch.float32, eb.EGG_F32, eb.EGG_NORMAL, 0),
                              "raw": (torch.int32, eb.EGG_U32, eb.EGG_RAW, 0), "int": (torch.int8, eb.EGG_I8, eb.EGG_UNIFORM_INT, 8),
                              "table": (torch.int8, eb.EGG_I8, eb.EGG_NORMAL_INT16, 0)}[dist]
    key, begin = eb.make_key(0x123456789, 4, 11), 2**32 - members  # the last member ids
    got = torch.empty((members, n, 1), dtype=tdt, device="cuda")
    longer = torch.empty((members, n + 1, 1), dtype=tdt, device="cuda")  # not whole pieces: the general kernel
    ctx.eggroll_noise_gen(key, eb.make_shape(begin, members, 1, n, n, 1), code, kind, bound, got, None)
    ctx.eggroll_noise_gen(key, eb.make_shape(begin, members, 1, n + 1, n, 1), code, kind, bound, longer, None)
    assert torch.equal(got.view(members, n), longer.view(members, n + 1)[:, :n])


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("rank", [1, 2, 4, 8, 16])
@pytest.mark.parametrize("members", [1, 3, 1024, 1025])  # a partial chunk; both sides of where each workgroup finds the norm itself
def test_generated_panels_equal_packed(ctx, dtype, rank, members):
    import torch
    tdt, code = (torch.bfloat16, eb.EGG_BF16) if dtype == "bf16" else (torch.float32, eb.EGG_F32)
    d_out, d_in = 132, 68 if rank == 1 else 67  # odd widths are taken from rank 2 on
    key, shape = eb.make_key(5, 1, 3), eb.make_shape(7, members, 1, d_out, d_in, rank)
    A = torch.empty((members, d_out, rank), dtype=tdt, device="cuda")
    B = torch.empty((members, d_in, rank), dtype=tdt, device="cuda")
    ctx.eggroll_noise_gen(key, shape, code, eb.EGG_NORMAL, 0, A, B)
    f = torch.randn(members, generator=torch.Generator("cuda").manual_seed(members), device="cuda") * 37.0
    G, H = (torch.empty((d_out, d_in), dtype=torch.float32, device="cuda") for _ in range(2))
    ctx.eggroll_update(key, shape, code, f, 0.25, 0, G, None, 0.0, A, B)
    ctx.eggroll_update(key, shape, code, f, 0.25, 0, H)
    assert G.abs().max() > 0 and torch.equal(G, H)


@pytest.mark.parametrize("rank", [1, 2, 4, 8, 16])
@pytest.mark.parametrize("d_out", [4096, 4092])  # (rank 1: the block form and the general one)
def test_panel_entries_are_rounded_as_stated(ctx, rank, d_out):
    """B picks one (member, rank term) per column of G, so G is the A panel itself, times a power of two: the product of the bf16 factor
    and the fp32 fitness rounded to fp16 once at rank 2, 4 and 8, after a rounding to fp32 at rank 1 and 16.  Exact."""
    import numpy as np
    import torch
    N = 64 // rank
    g = torch.Generator("cuda").manual_seed(rank)
    A = torch.randn((N, d_out, rank), generator=g, device="cuda").to(torch.bfloat16)
    B = torch.zeros((N, 64, rank), dtype=torch.bfloat16, device="cuda")
    i, l = np.divmod(np.arange(64), rank)
    B[i, np.arange(64), l] = 1.0
    # fitness values for which some 8-bit factor's product rounds to another fp16 value by way of fp32 (one in 130)
    draws = np.random.default_rng(rank).uniform(0.5, 1.0, 20000).astype(np.float32)
    exact = draws[:, None].astype(np.float64) * np.arange(128, 256)
    draws = draws[(exact.astype(np.float16) != exact.astype(np.float32).astype(np.float16)).any(1)]
    f = torch.from_numpy(draws[:N]).cuda()
    G = torch.empty((d_out, 64), device="cuda")
    ctx.eggroll_update(eb.make_key(1, 1, 1), eb.make_shape(0, N, 1, d_out, 64, rank), eb.EGG_BF16, f, 1.0, 0, G, None, 0.0, A, B)
    a, fit = A.float().cpu().numpy(), f.cpu().numpy()
    norm = 2.0 ** np.ceil(np.log2(np.abs(fit).max()))
    product = a[i, :, l].T.astype(np.float64) * (fit / norm).astype(np.float64)[i]
    want = (product if rank in (2, 4, 8) else product.astype(np.float32)).astype(np.float16)
    if rank in (2, 4, 8):
        assert (want != product.astype(np.float32).astype(np.float16)).any()  # the two do differ
    assert (G.cpu().numpy() == want.astype(np.float32) * norm).all()


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("rank", [2, 4, 8, 16])
@pytest.mark.parametrize("anti", [0, 1])
@pytest.mark.parametrize("d_in", [8, 264, 1032])
def test_one_row_projection(ctx, dtype, rank, anti, d_in):
    """One row per member at rank >= 2 (threads expand pieces and multiply at once), seen through a layer with zero weights:
    Y = c t A^T.  fp32 sums of d_in products and, in bf16, one rounding of Y: 1e-5 and 2^-8 of the row's size."""
    import torch
    tdt, code = (torch.bfloat16, eb.EGG_BF16) if dtype == "bf16" else (torch.float32, eb.EGG_F32)
    N, d_out = 6, 64
    g = torch.Generator("cuda").manual_seed(d_in)
    X = torch.randn((N, d_in), generator=g, device="cuda").to(tdt)
    W = torch.zeros((d_out, d_in), dtype=tdt, device="cuda")
    Y = torch.empty((N, d_out), dtype=tdt, device="cuda")
    ids = N // 2 if anti else N
    A = torch.empty((ids, d_out, rank), dtype=tdt, device="cuda")
    B = torch.empty((ids, d_in, rank), dtype=tdt, device="cuda")
    key, sigma = eb.make_key(8, 2, 1), 0.5
    ctx.eggroll_perturbed_forward(key, eb.make_shape(4, N, 1, d_out, d_in, rank, anti), sigma, eb.EGG_ACT_NONE, W, X, Y, A, B)
    A2, B2 = torch.empty_like(A), torch.empty_like(B)
    ctx.eggroll_noise_gen(key, eb.make_shape(4 // (2 if anti else 1), ids, 1, d_out, d_in, rank), code, eb.EGG_NORMAL, 0, A2, B2)
    assert torch.equal(A, A2) and torch.equal(B, B2)
    of = torch.arange(N, device="cuda") // (2 if anti else 1)
    t = (X.double()[:, :, None] * B.double()[of]).sum(1)
    if anti:
        t[1::2] *= -1
    ref = (t[:, None, :] * A.double()[of]).sum(-1) * (sigma / rank ** 0.5)
    tol = (1e-5 if dtype == "f32" else 2.0 ** -8) * (ref.abs() + ref.square().mean(1, keepdim=True).sqrt())
    assert ((Y.double() - ref).abs() <= tol).all()
