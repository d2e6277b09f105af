"""GPU: the map from bytes to integers, two bytes at a time, for every bound, in the generator of factors and in that of the update's
panels; exact against the oracle's map of the stream's bytes."""
import pytest

import oracle
from paper_2511_16652_amd import binding as eb

pytestmark = pytest.mark.gpu


def test_every_bound():
    import numpy as np
    import torch
    ctx = eb.Context(0)
    key, n = eb.make_key(9, 1, 4), 2048   # 2048 values of a member meet every byte (seen in the check below)
    seen = np.unique(oracle.raw_words(9, 1, 4, 0, 5, 0, n // 4).view(np.uint8))
    assert seen.size == 256
    A = torch.empty((1, n, 1), dtype=torch.int8, device="cuda")
    for bound in range(128):
        ctx.eggroll_noise_gen(key, eb.make_shape(5, 1, 1, n, n, 1), eb.EGG_I8, eb.EGG_UNIFORM_INT, bound, A, None)
        assert (A.cpu().numpy().ravel() == oracle.noise_int(9, 1, 4, 0, 5, 0, n, bound)).all(), bound
    torch.cuda.synchronize()
    ctx.close()
