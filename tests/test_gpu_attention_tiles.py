"""GPU: the causal attention kernel at the edges of its key blocks (32), of the 128 keys that sit in LDS at a time and of its query
block assignment, every head dimension.  Reference: softmax attention in 64 bits of the bf16 inputs; probabilities and outputs are
rounded to bf16 (2^-9 each, the first averaged over the keys): 1e-2 of |value| + rms."""
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


def reference(Q, K, V, N, S, heads):
    import torch
    hd = Q.shape[1] // heads
    q, k, v = (t.double().view(N, S, heads, hd).transpose(1, 2).contiguous().view(N * heads, S, hd) for t in (Q, K, V))
    s = torch.bmm(q, k.transpose(1, 2).contiguous()) / math.sqrt(hd)
    s.masked_fill_(torch.ones((S, S), dtype=torch.bool, device="cuda").triu(1), float("-inf"))
    o = torch.bmm(torch.softmax(s, -1), v)
    return o.view(N, heads, S, hd).transpose(1, 2).reshape(N * S, heads * hd)


@pytest.mark.parametrize("hd", [32, 64, 128])
@pytest.mark.parametrize("S", [1, 2, 31, 32, 33, 64, 95, 127, 128, 129, 160, 161, 200, 224, 225, 255, 256])
def test_tiles(ctx, hd, S):
    import torch
    N, heads = 3, 5
    g = torch.Generator("cuda").manual_seed(S)
    Q, K, V = (torch.randn((N * S, heads * hd), generator=g, device="cuda").to(torch.bfloat16) for _ in range(3))
    O = torch.full((N * S + 1, heads * hd), 7.0, dtype=torch.bfloat16, device="cuda")
    ctx.eggroll_causal_attention_bf16(N, S, heads, hd, Q * 2, K, V, O[:N * S])
    ref = reference(Q * 2, K, V, N, S, heads)
    assert ((O[:N * S].double() - ref).abs() <= 1e-2 * (ref.abs() + ref.square().mean().sqrt())).all()
    assert (O[N * S:] == 7.0).all()  # nothing is written past the last row


def test_an_infinite_value_stays_where_it_is_visible(ctx):
    """V of the last token of a ragged window is infinite in one column: that token's output is infinite there, and the rows before
    the key block it sits in are untouched."""
    import torch
    N, S, heads, hd = 2, 77, 2, 64
    g = torch.Generator("cuda").manual_seed(1)
    Q, K, V = (torch.randn((N * S, heads * hd), generator=g, device="cuda").to(torch.bfloat16) for _ in range(3))
    ref = reference(Q, K, V, N, S, heads)
    V[S - 1, 3] = float("inf")
    O = torch.empty_like(Q)
    ctx.eggroll_causal_attention_bf16(N, S, heads, hd, Q, K, V, O)
    assert torch.isposinf(O[S - 1, 3])
    keep = torch.ones_like(O, dtype=torch.bool)
    keep[64:S, 3] = False  # the key block of the last token
    assert ((O.double() - ref).abs()[keep] <= 1e-2 * (ref.abs()[keep] + ref.square().mean().sqrt())).all()


@pytest.mark.parametrize("hd", [32, 64, 128])
@pytest.mark.parametrize("S", [128, 129, 161, 200, 223, 256])
def test_members_do_not_depend_on_the_call(ctx, hd, S):
    """A member's rows and projections are the same bits whatever else is in the call: few (member, head) pairs run in workgroups of
    eight waves, more of them than compute units in workgroups of four.  The larger call is also held to the reference: it is the one
    that brings ragged windows to the kernel of four waves."""
    import torch
    N, heads = 90, 4
    g = torch.Generator("cuda").manual_seed(S + hd)
    Q, K, V = (torch.randn((N * S, heads * hd), generator=g, device="cuda").to(torch.bfloat16) for _ in range(3))
    key = eb.make_key(3, 1, 4)

    def run(first, n):
        q, k, v = (t[first * S:(first + n) * S].contiguous() for t in (Q * 2, K, V))
        o, t_next = torch.empty_like(q), torch.empty(n * S, device="cuda")
        ctx.eggroll_causal_attention_project_bf16(key, first, n, S, heads, hd, q, k, v, o, t_next)
        return o, t_next

    O, t = run(0, N)
    for first, n in ((0, 1), (41, 3), (N - 60, 60)):
        o, tn = run(first, n)
        assert torch.equal(o, O[first * S:(first + n) * S]) and torch.equal(tn, t[first * S:(first + n) * S]), (first, n)
    ref = reference(Q * 2, K, V, N, S, heads)
    assert ((O.double() - ref).abs() <= 1e-2 * (ref.abs() + ref.square().mean().sqrt())).all()
