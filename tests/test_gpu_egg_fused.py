"""GPU: the integer model in one kernel (D = 256), bit for bit against the oracle: around the numbers of rows of its workgroups and of the rule
between them, over the whole range of weights, biases, states and normalisation weights, and at the shifts where the pass-by-pass form
takes over."""
import numpy as np
import pytest

import oracle
from helpers import memory_left
from paper_2511_16652_amd import binding as eb

pytestmark = pytest.mark.gpu

SEED, STEP, LAYER, D = 21, 2, 5, 256


@pytest.fixture(scope="module")
def ctx():
    import torch
    c = eb.Context(0)
    yield c
    torch.cuda.synchronize()
    c.close()


@pytest.mark.parametrize("L,N,T,mb,anti,bound,cs", [
    (1, 1, 1, 0, 0, 8, 4), (2, 31, 3, 7, 0, 8, 4), (1, 32, 2, 0, 1, 8, 0), (2, 33, 1, 3, 0, 127, 4), (3, 98, 2, 6, 1, 8, 7), (0, 40, 2, 0, 0, 8, 4),
    (1, 8194, 2, 0, 1, 8, 4),                  # two workgroups of 32 rows on some CUs
    (1, 16386, 1, 2, 1, 8, 4), (1, 24575, 1, 1, 0, 3, 5),      # 96 rows
    (1, 24650, 2, 0, 1, 8, 4), (1, 32767, 1, 0, 0, 8, 4),      # 128 rows
    (1, 130, 2, 0, 1, "table", 4), (1, 24580, 1, 0, 0, "table", 4),   # the table's noise needs the 32-bit product
    (1, 2100, 2, 0, 1, 8, 8),                  # past the folded shifts of the 1024-wide product: pass by pass
])
def test_bit_exact(ctx, L, N, T, mb, anti, bound, cs):
    import torch
    rng = np.random.default_rng(N + cs)
    i8 = lambda lo, hi, *s: rng.integers(lo, hi + 1, s).astype(np.int8)  # noqa: E731
    w = lambda *s: np.clip(np.rint(16 * rng.standard_normal(s)), -127, 127).astype(np.int8)  # noqa: E731
    P = {"emb": i8(-127, 127, 256, D), "ln1": i8(-127, 127, L, D), "gru_w": w(L, 4, D, D), "gru_b": i8(-127, 127, L, 2, D), "ln2": i8(-127, 127, L, D),
         "mlp1": w(L, 4 * D, D), "mlp2": w(L, D, 4 * D), "ln_out": i8(-127, 127, D), "head": w(256, D)}
    tok, S = rng.integers(0, 256, (T, N)).astype(np.uint8), i8(-127, 127, L, N, D)
    b = eb.EGG_INT_NOISE_NORMAL16 if bound == "table" else bound
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()  # noqa: E731
    S_out = torch.full((L, N, D), 99, dtype=torch.int8, device="cuda")
    logits = torch.full((T, N, 256), 99, dtype=torch.int8, device="cuda")
    ctx.eggroll_egg_forward_i8(eb.make_key(SEED, STEP, LAYER), eb.make_shape(mb, N, 1, D, D, 1, antithetic=anti), L, b, cs, T,
                               {k: dev(v) for k, v in P.items()}, dev(tok), dev(S), S_out, logits)
    want, S_want = oracle.egg_forward_i8(SEED, STEP, LAYER, mb, N, D, L, b, cs, P, tok, S, antithetic=bool(anti))
    assert (S_out.cpu().numpy() == S_want).all()
    assert (logits.cpu().numpy() == want).all()


def test_little_memory():
    """The one kernel reads whole workgroups of factors and a copy of the weights in another order (here 550 MB, pass by pass 4 MB): without memory for
    them the call runs pass by pass, the same bits."""
    import torch
    L, N = 400, 2
    g = torch.Generator("cuda").manual_seed(1)
    i8 = lambda *s: torch.randint(-40, 41, s, generator=g, device="cuda", dtype=torch.int8)  # noqa: E731
    P = {"emb": i8(256, D), "ln1": i8(L, D), "gru_w": i8(L, 4, D, D), "gru_b": i8(L, 2, D), "ln2": i8(L, D), "mlp1": i8(L, 4 * D, D), "mlp2": i8(L, D, 4 * D),
         "ln_out": i8(D), "head": i8(256, D)}
    tok, S = torch.tensor([[3, 200]], dtype=torch.uint8, device="cuda"), i8(L, N, D)

    def forward():
        S_out, logits = torch.empty_like(S), torch.empty((1, N, 256), dtype=torch.int8, device="cuda")
        c = eb.Context(0)
        try:
            c.eggroll_egg_forward_i8(eb.make_key(SEED, STEP, LAYER), eb.make_shape(0, N, 1, D, D, 1), L, 8, 4, 1, P, tok, S, S_out, logits)
            torch.cuda.synchronize()
        finally:
            c.close()
        return S_out, logits

    want = forward()
    with memory_left(300 << 20):
        got = forward()
    assert all(torch.equal(a, b) for a, b in zip(got, want))
