"""The slot sort over several 256-token chunks, at the edges of its launch forms.

Up to 512 chunks every scatter workgroup sums the chunks' counts itself;
beyond, a scan launch does.  In a layer call the same kernels also quantize
the activations (workgroups beside the counting ones) and write the m-tile
table of the prefill GEMMs, so the fused layer is compared with the separate
calls, whose table comes from a kernel of its own.
"""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_cases import bf16_dev, quantize_weights_gpu, require_gpu, to_dev

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def moe():
    return require_gpu()


def _permute(moe, ids, e):
    t, k = ids.shape
    off = torch.full((e + 1,), -7, dtype=torch.int32, device="cuda")
    src = torch.full((t * k,), -7, dtype=torch.int32, device="cuda")
    dst = torch.full((t * k,), -7, dtype=torch.int32, device="cuda")
    st = torch.zeros(1, dtype=torch.int32, device="cuda")
    ws = torch.empty(moe.moe_permute_workspace(t, k, e), dtype=torch.uint8, device="cuda")
    moe.moe_permute(to_dev(ids), e, off, src, dst, st, ws)
    return off.cpu().numpy(), src.cpu().numpy(), dst.cpu().numpy(), int(st.item())


def _distinct_ids(rng, t, k, e):
    return np.argsort(rng.random((t, e)), axis=1)[:, :k].astype(np.int32)


@pytest.mark.parametrize("t,k,e", [(512, 1, 1), (513, 3, 5), (1000, 32, 33), (300, 7, 1024), (512 * 256, 2, 3),
                                   (512 * 256 + 1, 2, 3)], ids=lambda v: str(v))
def test_sort_over_chunks_equals_oracle(moe, t, k, e):
    ids = _distinct_ids(np.random.default_rng(t + e), t, k, e)
    off, src, dst, st = _permute(moe, ids, e)
    r_off, r_src, r_dst = oracle.permute(ids, e)
    assert st == 0
    assert np.array_equal(off, r_off) and np.array_equal(src, r_src) and np.array_equal(dst, r_dst)


@pytest.mark.parametrize("t", [257, 1025, 512 * 256 + 300])
def test_sort_over_chunks_parks_bad_slots(moe, t):
    """Bad slots in the first, a middle and the last chunk go after the valid rows, in slot order."""
    rng = np.random.default_rng(t)
    e, k = 9, 3
    ids = _distinct_ids(rng, t, k, e)
    valid = np.ones((t, k), bool)
    for tok in (0, 5, t // 2, t - 1):
        ids[tok, 1] = e + 3 if tok % 2 else -1
        valid[tok, 1] = False
    for tok in (2, t - 2):
        ids[tok, 2] = ids[tok, 0]
        valid[tok, 2] = False
    off, src, dst, st = _permute(moe, ids, e)
    assert st == (moe.MOE_DEV_BAD_EXPERT_ID | moe.MOE_DEV_DUP_EXPERT_ID)
    flat, good = ids.reshape(-1), np.flatnonzero(valid.reshape(-1))
    want = np.concatenate([good[np.argsort(flat[good], kind="stable")], np.flatnonzero(~valid.reshape(-1))])
    assert np.array_equal(src, want)
    assert np.array_equal(dst[src], np.arange(t * k))
    assert np.array_equal(off, np.searchsorted(np.sort(flat[good]), np.arange(e + 1)))


@pytest.mark.parametrize("t,zipf", [(65, 0.0), (255, 1.2), (700, 0.0), (1500, 1.5)])
def test_layer_tiles_from_the_sort_equal_the_separate_calls(moe, t, zipf):
    w = synth.Workload("chunks", 256, 128, 12, 3, t, "zipf" if zipf else "uniform", zipf, "sigmoid", seed=t)
    x = bf16_dev(synth.activations(w))
    ids, wts = (to_dev(a) for a in synth.routing(w))
    dw = quantize_weights_gpu(moe, *synth.weights_host(w))
    outs = []
    for fused in (True, False):
        buf = moe.MoELayerBuffers(256, 128, 12, 3, t, moe.MOE_REGIME_PREFILL, fused=fused)
        moe.run_layer(buf, x, ids, wts, dw)
        outs.append(buf.out.cpu().numpy())
        assert int(buf.dev_status.item()) == 0
    assert np.array_equal(*outs)


def _bad_ids(rng, t, k, e, share):
    """Distinct ids, of which `share` become -1, e or above, or the token's first id."""
    ids = _distinct_ids(rng, t, k, e)
    how = rng.integers(0, 3, (t, k))
    bad = np.where(how == 0, -1, np.where(how == 1, e + rng.integers(0, 9, (t, k)), ids[:, :1])).astype(np.int32)
    return np.where(rng.random((t, k)) < share, bad, ids)


@pytest.mark.parametrize("share", [0.01, 0.5, 1.0])
@pytest.mark.parametrize("t,k,e", [(256, 32, 40), (200, 7, 1024), (700, 8, 64), (2049, 1, 5), (512 * 256 + 300, 2, 3)])
def test_sort_parks_many_bad_slots(moe, t, k, e, share):
    ids = _bad_ids(np.random.default_rng(t + k), t, k, e, share)
    off, src, dst, _ = _permute(moe, ids, e)
    valid = (ids >= 0) & (ids < e)
    for j in range(1, k):
        valid[:, j] &= np.all(ids[:, :j] != ids[:, j:j + 1], axis=1)
    flat, good = ids.reshape(-1), np.flatnonzero(valid.reshape(-1))
    want = np.concatenate([good[np.argsort(flat[good], kind="stable")], np.flatnonzero(~valid.reshape(-1))])
    assert np.array_equal(src, want)
    assert np.array_equal(dst[src], np.arange(t * k))
    assert np.array_equal(off, np.searchsorted(np.sort(flat[good]), np.arange(e + 1)))


@pytest.mark.parametrize("t,k,e", [(256, 32, 1024), (8192, 8, 256)])
def test_bad_slots_are_not_walked_one_by_one(moe, t, k, e):
    """A rank's ids of other ranks' experts are -1: they must not make the sort many times slower."""
    ids = _distinct_ids(np.random.default_rng(0), t, k, e)
    half = np.where(np.random.default_rng(1).random((t, k)) < 0.5, -1, ids).astype(np.int32)
    times = []
    for a in (ids, half):
        d = to_dev(a)
        off = torch.empty(e + 1, dtype=torch.int32, device="cuda")
        src, dst = (torch.empty(t * k, dtype=torch.int32, device="cuda") for _ in range(2))
        ws = torch.empty(moe.moe_permute_workspace(t, k, e), dtype=torch.uint8, device="cuda")
        spans = []
        for _ in range(12):
            ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
            ev[0].record()
            for _ in range(10):
                moe.moe_permute(d, e, off, src, dst, None, ws)
            ev[1].record()
            ev[1].synchronize()
            spans.append(ev[0].elapsed_time(ev[1]))
        times.append(min(spans))
    # Measured: 9.5 -> 38 us and 10.5 -> 20 us; walked by one thread of each chunk 5590 and 486 us.
    assert times[1] < 10 * times[0]
