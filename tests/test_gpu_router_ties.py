"""The gate's selection rounds on equal keys, and the tiled logits at single and half steps.

Equal keys go to the lower expert: experts that share a router row have
bit-equal logits on the GPU too, so the choice among them is exact.  The
distinct rows' keys are far apart (the inputs are small integers, whose dot
products are exact in fp32), so every id must equal the oracle's.
"""
import numpy as np
import pytest
import torch

import synth
from gpu_cases import require_gpu, to_dev
from oracle import router_oracle as ro

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def moe():
    return require_gpu()


def _route(moe, x, wr, bias, k, n_group, kept, shared=-1):
    t = x.shape[0]
    cols = k + (shared >= 0)
    ids = torch.full((t, cols), -1, dtype=torch.int32, device="cuda")
    wts = torch.zeros((t, cols), dtype=torch.float32, device="cuda")
    ws = torch.empty(max(1, moe.moe_router_workspace(t, x.shape[1], wr.shape[0])), dtype=torch.uint8, device="cuda")
    moe.moe_router(to_dev(x.view(np.int16)), to_dev(wr.view(np.int16)), None if bias is None else to_dev(bias), ids,
                   wts, n_group, kept, 1.5, ws, shared_expert=shared)
    return ids.cpu().numpy(), wts.cpu().numpy()


# (tokens, experts, k, groups, kept): one token per workgroup and four; one to
# sixteen experts per lane; ragged expert counts; the largest k of the rounds.
@pytest.mark.parametrize("t,e,k,groups,kept", [(3, 64, 16, 1, 1), (3, 256, 8, 8, 4), (70, 7, 7, 1, 1),
                                               (70, 130, 16, 2, 1), (300, 256, 8, 8, 4), (300, 1024, 5, 64, 3)])
@pytest.mark.parametrize("offset", [0.0, -3.0])
def test_equal_keys_go_to_the_lower_expert(moe, t, e, k, groups, kept, offset):
    h = 256
    rng = np.random.default_rng(e + t)
    rows = np.zeros((3, h), np.float32)
    rows[0, :8], rows[1, 8:16], rows[2, 16:24] = 0.25, 0.25, 0.25
    x = np.zeros((t, h), np.float32)
    x[:, :24] = rng.permuted(np.repeat([[-1.0, 0.5, 1.5]], t, axis=0), axis=1).repeat(8, axis=1)
    wr = rows[rng.integers(0, 3, e)]
    bias = np.full(e, offset, np.float32)  # negative keys keep their order
    xb, wb = synth.bf16_bits_from_f32(x), synth.bf16_bits_from_f32(wr)
    ids, wts = _route(moe, xb, wb, bias, k, groups, kept)
    want_ids, want_w = ro.router(xb, wb, bias, k, groups, kept, 1.5)
    assert np.array_equal(ids, want_ids)
    assert np.allclose(wts, want_w, rtol=0, atol=1e-5 * 1.5)  # the gate's bound on its 32-bit weights


@pytest.mark.parametrize("hidden", [32, 64, 96, 160, 192, 224])
@pytest.mark.parametrize("t", [256, 385])
def test_tiled_logits_of_few_steps(moe, hidden, t):
    """One to four 64-K steps, the last one whole or half, on the tiled kernel
    (256 tokens or more), with a ragged last token tile and 48 of 256 experts."""
    rng = np.random.default_rng(hidden + t)
    e, k = 48, 4
    x = synth.bf16_bits_from_f32(rng.integers(-4, 5, (t, hidden)).astype(np.float32) / 8)
    wr = synth.bf16_bits_from_f32(rng.integers(-8, 9, (e, hidden)).astype(np.float32) / 16)
    ids, wts = _route(moe, x, wr, None, k, 1, 1, shared=e)
    want_ids, want_w = ro.router(x, wr, None, k, 1, 1, 1.5)
    # The logits are exact (multiples of 2^-7 below 2^7).  Distinct ones differ
    # by at least that, but their 32-bit sigmoids may round to the same or to
    # neighbouring values in another order where they saturate: those tokens out.
    s = np.sort(ro.router(x, wr, None, k, 1, 1, 1.5, want_intermediates=True)[2]["scores"], axis=1)[:, ::-1][:, :k + 1]
    gap = s[:, :-1] - s[:, 1:]
    clear = np.all((gap == 0) | (gap > 1e-6), axis=1) & (s[:, 0] < 1 - 1e-6)
    assert clear.mean() > 0.5
    assert np.array_equal(ids[clear, :k], want_ids[clear])
    assert np.allclose(wts[clear, :k], want_w[clear], rtol=0, atol=1e-5 * 1.5)
    assert np.all(ids[:, k] == e) and np.all(wts[:, k] == 1.0)


@pytest.mark.parametrize("t", [256, 768, 769])
@pytest.mark.parametrize("e", [40, 300])
def test_tiled_logits_around_the_tile_order(moe, t, e):
    """Up to six 128-token tiles are the fastest grid index, beyond them the K slices; one and two expert tiles."""
    rng = np.random.default_rng(e + t)
    k = 4
    x = synth.bf16_bits_from_f32(rng.integers(-4, 5, (t, 1024)).astype(np.float32) / 8)
    wr = synth.bf16_bits_from_f32(rng.integers(-8, 9, (e, 1024)).astype(np.float32) / 64)
    ids, wts = _route(moe, x, wr, None, k, 1, 1)
    want_ids, want_w = ro.router(x, wr, None, k, 1, 1, 1.5)
    # Exact logits (multiples of 2^-9 below 2^6); tokens whose rounded sigmoids are as close as above are left out.
    s = np.sort(ro.router(x, wr, None, k, 1, 1, 1.5, want_intermediates=True)[2]["scores"], axis=1)[:, ::-1][:, :k + 1]
    gap = s[:, :-1] - s[:, 1:]
    clear = np.all((gap == 0) | (gap > 1e-6), axis=1)
    assert clear.mean() > 0.5
    assert np.array_equal(ids[clear], want_ids[clear])
    assert np.allclose(wts[clear], want_w[clear], rtol=0, atol=1e-5 * 1.5)


@pytest.mark.parametrize("nan", [0x7fc00000, 0xffc00000], ids=["plus", "minus"])
@pytest.mark.parametrize("t", [1, 70, 300])
def test_nan_keys_come_last(moe, t, nan):
    """An expert whose key is NaN (a NaN in its bias or router row, of either sign) is chosen by no token while
    there are others; a token of NaNs takes the lowest experts, each once."""
    rng = np.random.default_rng(t)
    h, e, k, bad = 256, 70, 8, 66
    x = rng.integers(-4, 5, (t, h)).astype(np.float32) / 8
    wr = rng.integers(-8, 9, (e, h)).astype(np.float32) / 64
    xb, wb = synth.bf16_bits_from_f32(x), synth.bf16_bits_from_f32(wr)
    want, _ = ro.router(xb, np.delete(wb, bad, 0), None, k)
    want = want + (want >= bad)
    bias = np.zeros(e, np.float32)
    bias.view(np.uint32)[bad] = nan
    row = wb.copy()
    row[bad, 3] = nan >> 16
    for ids, wts in (_route(moe, xb, wb, bias, k, 1, 1), _route(moe, xb, row, None, k, 1, 1)):
        assert np.array_equal(ids, want)
        assert np.all(np.isfinite(wts))
    xb[t // 2] = nan >> 16
    ids, wts = _route(moe, xb, wb, None, k, 1, 1)
    assert np.array_equal(ids[t // 2], np.arange(k)) and np.all(np.isnan(wts[t // 2]))
