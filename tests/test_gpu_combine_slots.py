"""The combine's slot batches (8 at a time, then the remaining 1 to 7 in one) at every remainder, bit for bit."""
import numpy as np
import pytest
import torch

import oracle
from gpu_cases import require_gpu, to_dev

pytestmark = pytest.mark.gpu


# Columns: less than one wave, one wave's 256, a workgroup's 1024, one block more.
@pytest.mark.parametrize("h", [128, 256, 1024, 1152])
@pytest.mark.parametrize("k", [1, 2, 3, 4, 5, 6, 7, 8, 9, 15, 16, 31])
def test_combine_every_slot_count(k, h):
    moe = require_gpu()
    rng = np.random.default_rng(100 * k + h)
    t = 5
    y = (rng.standard_normal((t * k, h)) * np.exp(rng.uniform(-20, 20, (t * k, 1)))).astype(np.float32)
    dest = rng.permutation(t * k).astype(np.int32)
    wts = rng.random((t, k)).astype(np.float32)
    out = torch.empty((t + 1, h), dtype=torch.int16, device="cuda").fill_(-7)
    moe.moe_combine(to_dev(y), to_dev(dest), to_dev(wts), out[:t])
    got = out.cpu().numpy()
    assert np.array_equal(got[:t].view(np.uint16), oracle.combine(y, dest, wts))
    assert np.all(got[t] == -7)  # nothing past the last token
