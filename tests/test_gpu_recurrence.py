"""GPU: many time steps of the integer recurrent cell in one kernel, bit for bit against as many single steps (the general matmul
path, which test_gpu_int8 holds to the oracle): both sides of every register split of theta, ragged widths and row counts."""
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


@pytest.mark.parametrize("d", [16, 48, 256, 272, 512, 528, 768, 784, 1008, 1024])
@pytest.mark.parametrize("rows,anti", [(2, 1), (31, 0), (33, 0), (130, 1), (4098, 1)])
@pytest.mark.parametrize("bound,cs,steps", [(8, 4, 4), (127, 2, 5), (eb.EGG_INT_NOISE_NORMAL16, 6, 7)])
def test_steps_in_one_kernel_equal_single_steps(ctx, d, rows, anti, bound, cs, steps):
    import torch
    g = torch.Generator("cuda").manual_seed(d)
    W = torch.randint(-127, 128, (d, d), generator=g, device="cuda", dtype=torch.int8)
    H = torch.randint(-127, 128, (rows, d), generator=g, device="cuda", dtype=torch.int8)
    key, shape = eb.make_key(5, 6, 7), eb.make_shape(4, rows, 1, d, d, 1, anti)
    os = 4 + (d.bit_length() // 2)
    out = torch.empty_like(H)
    ctx.eggroll_perturbed_forward_i8(key, shape, bound, cs, os, steps, W, H, out)
    a, b = H.clone(), torch.empty_like(H)
    for _ in range(steps):
        ctx.eggroll_perturbed_forward_i8(key, shape, bound, cs, os, 1, W, a, b)
        a, b = b, a
    assert torch.equal(out, a) and (d < 48 or out.float().std() > 1)
    ctx.eggroll_perturbed_forward_i8(key, shape, bound, cs, os, steps, W, H, H)  # in place
    assert torch.equal(H, a)
