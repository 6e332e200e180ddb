"""The wide prefill tiles (256 expert rows) against the narrow ones and the oracle.

Both kernels compute each row with the same instructions in the same order, so
they agree bit for bit.  The narrow kernel takes a call whose row scales are not
16-byte aligned, which is how the same inputs run through both.  Every size here
has several hundred work items for the wide kernel's 256 workgroups, so most
tiles come from the queues; _wide asserts that the library takes wide tiles.
"""
import numpy as np
import pytest
import torch

import oracle
import synth
from gpu_cases import bits_to_f32, log, quantize_weights_gpu, rel_err, require_gpu, to_dev

pytestmark = pytest.mark.gpu

# Rows of the first three of four experts (the last takes the rest): tiles of 1
# to 8 row groups, odd and even, whole and ragged, one row.
SIZES = [(1, 289, 1023), (0, 31, 257), (65, 160, 1057), (224, 416, 448), (33, 128, 700), (2725, 2725, 2725)]
TOKENS = {4096: 10900, 4608: 13700}  # H -> tokens, one expert each, of four experts
TOKENS3 = {4096: 3700, 4608: 4700}  # three each


@pytest.fixture(scope="module")
def moe():
    return require_gpu()


@pytest.fixture(scope="module", params=[(4096, 2048), (4608, 1536)], ids=lambda p: f"H{p[0]}I{p[1]}")
def weights(moe, request):
    h, i = request.param
    w = synth.Workload("wide", h, i, 4, 1, TOKENS[h], "uniform", 0.0, "sigmoid", seed=h)
    host = synth.weights_host(w)
    return w, synth.activations(w), host, quantize_weights_gpu(moe, *host)


def _wide(moe, w, t, k=1, experts=4):
    """The launch takes wide tiles, of which most come from the queues."""
    dims = moe.MoeDims(w.hidden, w.inter, experts, k)
    assert moe.moe_prefill_tile_rows(dims, t) == 256
    items = t * k // 256 * min(w.inter // 128, w.hidden // 256)  # at least
    assert items >= 256 + 64, items


def _ids(sizes, t):
    ids = np.repeat(np.arange(4, dtype=np.int32), (*sizes, t - sum(sizes)))
    np.random.default_rng(sizes[0]).shuffle(ids)
    return ids[:, None]


def _ffn(moe, w, x, ids, dw, offset):
    """(y_rows, dest_row) of the prefill regime with sx `offset` floats into its buffer."""
    (t, h), k = x.shape, ids.shape[1]
    dims = moe.MoeDims(w.hidden, w.inter, w.n_experts, k)
    qx = torch.empty((t, h), dtype=torch.uint8, device="cuda")
    sx = torch.empty(t * (h // 128) + 4, dtype=torch.float32, device="cuda")[offset:offset + t * (h // 128)]
    moe.moe_quant_act(to_dev(x.view(np.int16)), qx, sx.view(t, h // 128))
    off = torch.empty(w.n_experts + 1, dtype=torch.int32, device="cuda")
    src, dst = (torch.empty(t * k, dtype=torch.int32, device="cuda") for _ in range(2))
    pws = torch.empty(moe.moe_permute_workspace(t, k, w.n_experts), dtype=torch.uint8, device="cuda")
    moe.moe_permute(to_dev(ids), w.n_experts, off, src, dst, None, pws)
    y = torch.full((t * k, h), float("nan"), dtype=torch.float32, device="cuda")
    ws = torch.empty(moe.moe_expert_ffn_workspace(dims, t, moe.MOE_REGIME_PREFILL), dtype=torch.uint8, device="cuda")
    moe.moe_expert_ffn(dims, t, moe.MOE_REGIME_PREFILL, qx, sx, off, src, *dw, y, ws)
    return y, dst


@pytest.mark.parametrize("sizes", SIZES, ids=lambda v: "_".join(map(str, v)))
def test_wide_tiles_equal_the_narrow_ones(moe, weights, sizes):
    w, x, _, dw = weights
    _wide(moe, w, w.tokens)
    y0, _ = _ffn(moe, w, x, _ids(sizes, w.tokens), dw, 0)
    y1, _ = _ffn(moe, w, x, _ids(sizes, w.tokens), dw, 1)
    assert torch.isfinite(y0).all()
    assert torch.equal(y0, y1)


def _layer(moe, w, x, ids, dw, wts=None, repeats=1):
    """Outputs of `repeats` layer calls on one workspace that holds no zeros before the first."""
    t, k = ids.shape
    buf = moe.MoELayerBuffers(w.hidden, w.inter, 4, k, t, moe.MOE_REGIME_PREFILL, fused=True)
    buf.layer_ws.fill_(0x7f)  # queue counters that a call did not clear would end its launches at once
    wts = torch.ones((t, k), device="cuda") if wts is None else wts
    return [moe.run_layer(buf, to_dev(x.view(np.int16)), to_dev(ids), wts, dw).clone() for _ in range(repeats)]


def test_wide_tiles_repeat_and_meet_the_oracle(moe, weights):
    """The work queues hand out tiles in another order every time: same bits.  The
    layer output against the oracle within the library's bound."""
    w, x, host, dw = weights
    _wide(moe, w, w.tokens)
    ids = _ids(SIZES[0], w.tokens)
    outs = _layer(moe, w, x, ids, dw, repeats=3)
    assert torch.equal(outs[0], outs[1]) and torch.equal(outs[0], outs[2])
    pick = np.concatenate([np.flatnonzero(ids[:, 0] == e)[[0, -1]] for e in range(4)])
    ref = oracle.moe_layer(x[pick], ids[pick], np.ones((len(pick), 1), np.float32), oracle.prepare_weights(*host))
    err = rel_err(bits_to_f32(outs[0][torch.from_numpy(pick).cuda()]), oracle.bf16_to_f32(ref))
    log(f"wide H={w.hidden} I={w.inter}: rel err {err:.3e}")
    assert err <= 2e-2


@pytest.mark.parametrize("left_out", [(0.25, 0.25, 0.25, 0.25), (0.0, 0.02, 0.28, 0.7), (0.97, 0.01, 0.01, 0.01)])
def test_wide_layer_of_three_experts_a_token(moe, weights, left_out):
    """Three slots a token, the fourth expert left out by the given shares (experts of a few rows to all tokens: the
    eight ranges of work items run dry at different times): the fused layer, whose sort clears the queues and
    writes the tile table, against the four calls with narrow tiles, three times on one workspace."""
    w, x, _, dw = weights
    t = TOKENS3[w.hidden]
    _wide(moe, w, t, k=3)
    rng = np.random.default_rng(t)
    out = rng.choice(4, t, p=left_out)
    ids = np.array([rng.permutation([e for e in range(4) if e != o]) for o in out], dtype=np.int32)
    wts = torch.rand((t, 3), device="cuda") + 0.1
    y, dst = _ffn(moe, w, x[:t], ids, dw, 1)
    want = torch.empty((t, w.hidden), dtype=torch.int16, device="cuda")
    moe.moe_combine(y, dst, wts, want)
    for got in _layer(moe, w, x[:t], ids, dw, wts, repeats=3):
        assert torch.equal(got, want)


@pytest.mark.parametrize("chunk", [2600, 5011])
def test_wide_tiles_over_chunks_equal_the_resident_layer(moe, weights, chunk):
    """Row tables: a streamed launch (two experts, half of the rows) has tiles that span chunks."""
    w, x, _, dw = weights
    t = w.tokens
    _wide(moe, w, t, experts=2)
    w, x = w.with_tokens(2 * t), np.concatenate([x, x[::-1]])
    ids = np.concatenate([_ids(SIZES[2], t), 3 - _ids(SIZES[0], t)])
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
    assert torch.equal(out, _layer(moe, w, x, ids, dw)[0])
