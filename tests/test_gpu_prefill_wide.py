"""The wide prefill tiles (256 expert rows) against the narrow ones and the oracle.

Both kernels compute each row with the same instructions in the same order, so
they agree bit for bit.  The narrow kernel takes a call whose row scales are not
16-byte aligned, which is how the same inputs run through both.
"""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_cases import bits_to_f32, log, quantize_weights_gpu, rel_err, require_gpu, to_dev

pytestmark = pytest.mark.gpu

# Expert sizes (2800 rows over four experts, for which the library takes wide
# tiles): tiles of 1 to 8 row groups, odd and even, whole and ragged, one row.
SIZES = [(1, 289, 1023, 1487), (0, 31, 257, 2512), (65, 160, 1057, 1518), (224, 416, 448, 1712), (33, 128, 700, 1939),
         (700, 700, 700, 700)]


@pytest.fixture(scope="module")
def moe():
    return require_gpu()


@pytest.fixture(scope="module", params=[(4096, 2048), (4608, 1536)], ids=lambda p: f"H{p[0]}I{p[1]}")
def weights(moe, request):
    h, i = request.param
    w = synth.Workload("wide", h, i, 4, 1, 2800, "uniform", 0.0, "sigmoid", seed=h)
    host = synth.weights_host(w)
    return w, synth.activations(w), host, quantize_weights_gpu(moe, *host)


def _ids(sizes):
    ids = np.repeat(np.arange(4, dtype=np.int32), sizes)
    np.random.default_rng(sizes[0]).shuffle(ids)
    return ids[:, None]


def _ffn(moe, w, x, ids, dw, offset):
    """y_rows of the prefill regime with sx `offset` floats into its buffer."""
    t, h = x.shape
    dims = moe.MoeDims(w.hidden, w.inter, w.n_experts, 1)
    qx = torch.empty((t, h), dtype=torch.uint8, device="cuda")
    sx = torch.empty(t * (h // 128) + 4, dtype=torch.float32, device="cuda")[offset:offset + t * (h // 128)]
    moe.moe_quant_act(to_dev(x.view(np.int16)), qx, sx.view(t, h // 128))
    off = torch.empty(w.n_experts + 1, dtype=torch.int32, device="cuda")
    src, dst = (torch.empty(t, dtype=torch.int32, device="cuda") for _ in range(2))
    pws = torch.empty(moe.moe_permute_workspace(t, 1, w.n_experts), dtype=torch.uint8, device="cuda")
    moe.moe_permute(to_dev(ids), w.n_experts, off, src, dst, None, pws)
    y = torch.full((t, h), float("nan"), dtype=torch.float32, device="cuda")
    ws = torch.empty(moe.moe_expert_ffn_workspace(dims, t, moe.MOE_REGIME_PREFILL), dtype=torch.uint8, device="cuda")
    moe.moe_expert_ffn(dims, t, moe.MOE_REGIME_PREFILL, qx, sx, off, src, *dw, y, ws)
    return y


@pytest.mark.parametrize("sizes", SIZES, ids=lambda v: "_".join(map(str, v)))
def test_wide_tiles_equal_the_narrow_ones(moe, weights, sizes):
    w, x, _, dw = weights
    y0 = _ffn(moe, w, x, _ids(sizes), dw, 0)
    y1 = _ffn(moe, w, x, _ids(sizes), dw, 1)
    assert torch.isfinite(y0).all()
    assert torch.equal(y0, y1)


def _layer(moe, w, x, ids, dw):
    buf = moe.MoELayerBuffers(w.hidden, w.inter, 4, 1, w.tokens, moe.MOE_REGIME_PREFILL, fused=True)
    moe.run_layer(buf, to_dev(x.view(np.int16)), to_dev(ids), torch.ones((w.tokens, 1), device="cuda"), dw)
    return buf.out


def test_wide_tiles_repeat_and_meet_the_oracle(moe, weights):
    """The work queues hand out tiles in another order every time: same bits.  The
    layer output against the oracle within the library's bound."""
    w, x, host, dw = weights
    ids = _ids(SIZES[0])
    outs = [_layer(moe, w, x, ids, dw) for _ in range(3)]
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
    pick = np.concatenate([np.flatnonzero(ids[:, 0] == e)[[0, -1]] for e in range(4)])
    ref = oracle.moe_layer(x[pick], ids[pick], np.ones((len(pick), 1), np.float32), oracle.prepare_weights(*host))
    err = rel_err(bits_to_f32(outs[0][torch.from_numpy(pick).cuda()]), oracle.bf16_to_f32(ref))
    log(f"wide H={w.hidden} I={w.inter}: rel err {err:.3e}")
    assert err <= 2e-2


@pytest.mark.parametrize("chunk", [700, 1311])
def test_wide_tiles_over_chunks_equal_the_resident_layer(moe, weights, chunk):
    """Row tables: a streamed launch (two experts, 2800 rows) has tiles that span chunks."""
    w, x, _, dw = weights
    w, x, ids = w.with_tokens(5600), np.concatenate([x, x[::-1]]), np.concatenate([_ids(SIZES[2]), _ids(SIZES[0])])
    dims = moe.MoeDims(w.hidden, w.inter, 4, 1)
    host = []
    for m in dw:
        p = torch.empty(m.shape, dtype=m.dtype, pin_memory=True)
        p.copy_(m)
        host.append(p)
    ctx = moe.StreamContext(4)
    ring = torch.empty(moe.moe_ring_bytes(dims, 4), dtype=torch.uint8, device="cuda")
    ring_s = torch.empty(moe.moe_ring_scale_bytes(dims, 4) // 4, dtype=torch.float32, device="cuda")
    ws = torch.empty(moe.moe_ffn_streamed_workspace(dims, w.tokens, chunk), dtype=torch.uint8, device="cuda")
    out = torch.empty((w.tokens, w.hidden), dtype=torch.int16, device="cuda")
    copy = torch.cuda.Stream()
    moe.moe_ffn_streamed(dims, chunk, to_dev(x.view(np.int16)), to_dev(ids), torch.ones((w.tokens, 1), device="cuda"),
                         tuple(host), ring, ring_s, ctx, out, None, ws, torch.cuda.current_stream(), copy)
    torch.cuda.synchronize()
    ctx.close()
    assert torch.equal(out, _layer(moe, w, x, ids, dw))
