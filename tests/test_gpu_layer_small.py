"""The fused down + combine beyond 16 rows (small experts): edges of its rule, against the separate calls.

The fused layer must equal the four calls bit for bit: the same per-expert
arithmetic, K parts and combine order, whatever the launch form.
"""
import numpy as np
import pytest
import torch

import synth
from gpu_cases import bf16_dev, quantize_weights_gpu, require_gpu, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def moe():
    return require_gpu()


def _both(moe, h, i, e, k, t, routing, bad=()):
    w = synth.Workload("small", h, i, e, k, t, routing, 1.3 if routing == "zipf" else 0.0, "sigmoid", seed=t + k)
    x, (ids, wts) = synth.activations(w), synth.routing(w)
    ids = ids.copy()
    for tok, slot, value in bad:
        ids[tok, slot] = value
    dw = quantize_weights_gpu(moe, *synth.weights_host(w))
    bufs = []
    for fused in (True, False):
        buf = moe.MoELayerBuffers(h, i, e, k, t, moe.MOE_REGIME_DECODE, fused=fused)
        moe.run_layer(buf, bf16_dev(x), to_dev(ids), to_dev(wts), dw)
        bufs.append((buf.out.cpu().numpy(), int(buf.dev_status.item())))
    return bufs


@pytest.mark.parametrize("case", [
    (256, 128, 8, 2, 9, "uniform"),      # 18 rows
    (256, 128, 8, 2, 16, "zipf"),        # the token limit
    (256, 128, 8, 2, 17, "uniform"),     # beyond it: separate launches
    (512, 128, 16, 4, 16, "zipf"),       # 64 rows, 32 KB of W_down a workgroup
    (512, 256, 16, 4, 16, "uniform"),    # 64 rows, 64 KB: separate
    (256, 128, 300, 4, 16, "uniform"),   # more than 256 experts (rows of one), separate by the bytes
    (256, 128, 1024, 20, 1, "uniform"),  # one token with 20 slots
    (4096, 512, 4, 4, 16, "uniform"),    # full width: R * I at its limit, every expert 16 rows
    (4096, 640, 260, 3, 7, "zipf"),      # five K blocks over four parts, 21 rows, more than 256 experts
], ids=lambda c: "x".join(map(str, c)))
def test_small_layers_equal_the_separate_calls(moe, case):
    (a, sa), (b, sb) = _both(moe, *case)
    assert sa == sb == 0
    assert np.array_equal(a, b)


@pytest.mark.parametrize("h,i,e,k,t", [(256, 128, 8, 2, 16), (4096, 256, 8, 4, 12)])
def test_small_layers_with_bad_ids(moe, h, i, e, k, t):
    """Bad slots get no row: the tokens without one still equal the separate calls."""
    bad = [(1, 1, e + 5), (4, 0, -1)]
    (a, sa), (b, sb) = _both(moe, h, i, e, k, t, "uniform", bad)
    assert sa == sb == moe.MOE_DEV_BAD_EXPERT_ID
    good = [tok for tok in range(t) if tok not in (1, 4)]
    assert np.array_equal(a[good], b[good])


# (H, I, E, k, T) -> fused: edges of the rule beyond 16 rows.  H 5120 has 320 workgroups for 256 CUs.
@pytest.mark.parametrize("h,i,e,k,t,fused", [
    (256, 128, 8, 2, 16, True),     # 32 KB or less of W_down a workgroup
    (2048, 768, 4, 2, 9, False),    # half the CUs idle
    (4096, 512, 8, 4, 16, True),    # short experts up to 64 rows
    (5120, 512, 8, 4, 16, False),   # uneven workgroups: up to R * I = 20480
    (5120, 512, 8, 4, 10, True),
    (4096, 1024, 4, 2, 9, True),    # R * I = 18432
    (4096, 1024, 4, 4, 5, False),   # 20480
    (6144, 768, 4, 2, 9, True),     # a last round of 128 workgroups
    (5120, 768, 4, 2, 9, False),    # of 64
    (5120, 1536, 4, 2, 9, False),
    (5120, 1536, 4, 2, 8, True),    # 16 rows: always
])
def test_which_small_layers_are_fused(moe, h, i, e, k, t, fused):
    def matrices(r, c):
        return (torch.zeros((e, r, c), dtype=torch.uint8, device="cuda"),
                torch.ones((e, r // 128, c // 128), dtype=torch.float32, device="cuda"))

    ids = torch.arange(t * k, dtype=torch.int32, device="cuda").remainder(e).view(t, k)
    buf = moe.MoELayerBuffers(h, i, e, k, t, moe.MOE_REGIME_DECODE, fused=True)
    moe.moe_profile_begin(32)
    moe.run_layer(buf, torch.zeros((t, h), dtype=torch.int16, device="cuda"), ids, torch.ones((t, k), device="cuda"),
                  (*matrices(i, h), *matrices(i, h), *matrices(h, i)))
    names = [name for name, _ in moe.moe_profile_end()]
    assert ("ffn_decode_down_combine" in names) == fused and ("combine" in names) != fused
