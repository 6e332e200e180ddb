"""The workloads of this library whose time counts: routed-expert MoE layers, the gate and the streamed layer.

Each case is one call (or the fixed sequence of calls) that an inference
engine makes for one layer, through the package's entry points, on inputs
drawn from a seed: expert weights as a DeepSeek-V3 style FP8 checkpoint holds
them (e4m3 codes with one fp32 scale per 128 x 128 block), packed once by
``moe_pack_weight``; bf16 activations; router ids and weights.

Kinds of case:

* ``layer``    ``run_layer`` on fused buffers (``moe_ffn_layer``): a decode step
               of a few tokens, a batched decode step, a prefill chunk.
* ``steps``    the four calls of the layer (quantize, permute, expert FFN,
               combine), for engines that place work between them.
* ``w8a16``    ``run_layer`` with bf16 activations (decode only).
* ``router``   ``moe_router``: the gate in front of the layer.
* ``streamed`` ``moe_ffn_streamed``: the weights in pinned host memory.

``exact`` states the same definitions in plain torch, with every sum in 64
bits; the e4m3 quantizations of the activations and of SiLU(gate) * up are
part of the definition and are kept.
"""
import math

import torch

import paper_2606_10493_amd as moe

BLOCK = 128
E4M3_MAX = 448.0

# (hidden, expert intermediate, experts, experts per token)
DEEPSEEK_V3 = (7168, 2048, 256, 8)     # the model the library targets
SMALL_EXPERTS = (2048, 768, 128, 8)    # a mid-size MoE with narrow experts
FEW_EXPERTS = (4096, 1536, 16, 2)      # few, wide experts
TINY = (256, 128, 8, 2)                # the tests' tiny layer


def _case(name, kind, dims, tokens, zipf=0.0, **more):
    h, i, e, k = dims
    case = {"kind": kind, "hidden": h, "inter": i, "experts": e, "topk": k, "tokens": tokens, "zipf": zipf, **more}
    return {"name": name, **case} if name else case


def listed():
    return [
        # The smallest call: all launches and latency.
        _case("layer_tiny_16", "layer", TINY, 16),
        # Single-user decode: one token, eight experts' weights.
        _case("layer_decode_1", "layer", DEEPSEEK_V3, 1),
        # Decode with speculation or a handful of users.
        _case("layer_decode_4", "layer", DEEPSEEK_V3, 4),
        # A decode batch whose users share popular experts.
        _case("layer_decode_64_zipf", "layer", DEEPSEEK_V3, 64, 1.0),
        # A continuous-batching step (decodes and a short prompt), a ragged size.
        _case("layer_batch_201", "layer", DEEPSEEK_V3, 201),
        # A model with narrow experts, one short prompt.
        _case("layer_small_experts_509", "layer", SMALL_EXPERTS, 509, 0.6),
        # A prompt of about a thousand tokens, through the separate calls.
        _case("steps_prefill_1023", "steps", DEEPSEEK_V3, 1023, 0.4),
        # A full prefill chunk.
        _case("layer_prefill_8192", "layer", DEEPSEEK_V3, 8192),
        # bf16 activations, a few users.
        _case("w8a16_decode_5", "w8a16", DEEPSEEK_V3, 5),
        # The gate of a decode step and of a prefill chunk.
        _case("router_1", "router", DEEPSEEK_V3, 1, groups=8, kept=4, biased=True),
        _case("router_8192", "router", DEEPSEEK_V3, 8192, groups=8, kept=4, biased=True),
        # A layer streamed from host memory (a quarter of the experts of a
        # model that does not fit, two token chunks, a ring of half of them).
        _case("streamed_2048", "streamed", (7168, 2048, 32, 8), 2048, 0.8, chunk=1024, ring=16),
    ]


def _spread(rng, lo, hi):
    return max(lo, min(hi, round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))))


def draw(rng):
    kind = rng.choice(["layer", "layer", "layer", "layer", "layer", "steps", "w8a16", "router", "streamed"])
    zipf = rng.choice([0.0, 0.0, round(rng.uniform(0.2, 1.1), 2)])
    if kind in ("layer", "steps"):
        dims = rng.choice([DEEPSEEK_V3, DEEPSEEK_V3, SMALL_EXPERTS, FEW_EXPERTS])
        return _case(None, kind, dims, _spread(rng, 1, 8192), zipf)
    if kind == "w8a16":
        return _case(None, kind, rng.choice([DEEPSEEK_V3, SMALL_EXPERTS]), _spread(rng, 1, 64), zipf)
    if kind == "router":
        if rng.random() < 0.5:
            return _case(None, kind, DEEPSEEK_V3, _spread(rng, 1, 16384), groups=8, kept=4, biased=True)
        return _case(None, kind, SMALL_EXPERTS, _spread(rng, 1, 16384), groups=1, kept=1, biased=False)
    ring = rng.choice([2, 8, 16])
    return _case(None, kind, (7168, 2048, rng.choice([16, 24, 32]), 8), _spread(rng, 256, 2048), zipf,
                 chunk=rng.choice([512, 1024, 2048]), ring=ring)


# ------------------------------------------------------------------ inputs

def _gen(seed, which):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed * 16 + which)
    return g


def _fp8_matrices(g, n, rows, cols):
    """n matrices N(0, 0.02) quantized per 128 x 128 block: codes uint8 [n, rows, cols], scales fp32."""
    codes = torch.empty((n, rows, cols), dtype=torch.uint8, device="cuda")
    scales = torch.empty((n, rows // BLOCK, cols // BLOCK), dtype=torch.float32, device="cuda")
    step = max(1, (1 << 28) // (rows * cols))
    for a in range(0, n, step):
        b = min(n, a + step)
        w = torch.randn((b - a, rows // BLOCK, BLOCK, cols // BLOCK, BLOCK), generator=g, device="cuda").mul_(0.02)
        s = torch.maximum(w.amax((2, 4), keepdim=True), -w.amin((2, 4), keepdim=True)) / E4M3_MAX
        codes[a:b] = w.div_(s).to(torch.float8_e4m3fn).view(torch.uint8).view(b - a, rows, cols)
        scales[a:b] = s[:, :, 0, :, 0]
    return codes, scales


def _weights(case, seed):
    """(gate, s_gate, up, s_up, down, s_down), row-major codes, as a checkpoint holds them."""
    h, i, e = case["hidden"], case["inter"], case["experts"]
    out = []
    for which, (rows, cols) in enumerate(((i, h), (i, h), (h, i))):
        out += _fp8_matrices(_gen(seed, which), e, rows, cols)
    return out


def _packed(case, seed):
    w = _weights(case, seed)
    for j in (0, 2, 4):
        packed = torch.empty_like(w[j])
        moe.moe_pack_weight(w[j], packed)
        w[j] = packed
    return tuple(w)


def _tokens(case, seed):
    return torch.randn((case["tokens"], case["hidden"]), generator=_gen(seed, 4), device="cuda").to(torch.bfloat16)


def _routing(case, seed):
    """k distinct experts a token (popularity uniform or Zipf, in draw order) and normalised sigmoid weights."""
    g = _gen(seed, 5)
    t, e, k = case["tokens"], case["experts"], case["topk"]
    logp = -case["zipf"] * torch.log(torch.arange(1, e + 1, device="cuda", dtype=torch.float32))
    logp = logp[torch.randperm(e, generator=g, device="cuda")]
    u = torch.rand((t, e), generator=g, device="cuda").clamp_(1e-12, 1.0 - 1e-7)
    ids = torch.topk(logp - torch.log(-torch.log(u)), k, dim=1).indices.to(torch.int32).contiguous()
    w = torch.sigmoid(torch.randn((t, k), generator=g, device="cuda"))
    return ids, (w / w.sum(1, keepdim=True)).contiguous()


def _gate(case, seed):
    g = _gen(seed, 6)
    w = torch.randn((case["experts"], case["hidden"]), generator=g, device="cuda").mul_(0.02).to(torch.bfloat16)
    bias = torch.randn((case["experts"],), generator=g, device="cuda").mul_(0.02) if case["biased"] else None
    return w, bias


def prepare(case, seed):
    kind, t = case["kind"], case["tokens"]
    h, i, e, k = case["hidden"], case["inter"], case["experts"], case["topk"]
    x = _tokens(case, seed)
    if kind == "router":
        w, bias = _gate(case, seed)
        ws = torch.empty(max(256, moe.moe_router_workspace(t, h, e)), dtype=torch.uint8, device="cuda")
        ids = torch.empty((t, k), dtype=torch.int32, device="cuda")
        wts = torch.empty((t, k), dtype=torch.float32, device="cuda")
        return {"case": case, "x": x, "w": w, "bias": bias, "ids": ids, "wts": wts, "ws": ws}
    ids, wts = _routing(case, seed)
    state = {"case": case, "x": x, "ids": ids, "wts": wts}
    if kind != "streamed":
        state["weights"] = _packed(case, seed)
        state["buf"] = moe.MoELayerBuffers(h, i, e, k, t, fused=kind == "layer", w8a16=kind == "w8a16")
        return state
    host = []
    for m in _packed(case, seed):
        p = torch.empty(m.shape, dtype=m.dtype, pin_memory=True)
        p.copy_(m)
        host.append(p)
    dims, ring = moe.MoeDims(h, i, e, k), case["ring"]
    state["host"] = tuple(host)
    state["dims"] = dims
    state["ring"] = torch.empty(moe.moe_ring_bytes(dims, ring), dtype=torch.uint8, device="cuda")
    state["ring_scales"] = torch.empty(moe.moe_ring_scale_bytes(dims, ring) // 4, dtype=torch.float32, device="cuda")
    state["ctx"] = moe.StreamContext(ring)
    state["out"] = torch.empty((t, h), dtype=torch.int16, device="cuda")
    state["status"] = torch.zeros(1, dtype=torch.int32, device="cuda")
    state["ws"] = torch.empty(moe.moe_ffn_streamed_workspace(dims, t, case["chunk"]), dtype=torch.uint8, device="cuda")
    state["copy"] = torch.cuda.Stream()
    return state


# --------------------------------------------------------------------- run

def run(state):
    case = state["case"]
    if case["kind"] == "router":
        moe.moe_router(state["x"], state["w"], state["bias"], state["ids"], state["wts"], case["groups"], case["kept"],
                       2.5, ws=state["ws"])
        return {"ids": state["ids"], "weights": state["wts"]}
    if case["kind"] == "streamed":
        moe.moe_ffn_streamed(state["dims"], case["chunk"], state["x"], state["ids"], state["wts"], state["host"],
                             state["ring"], state["ring_scales"], state["ctx"], state["out"], state["status"],
                             state["ws"], copy_stream=state["copy"])
        return {"out": state["out"].view(torch.bfloat16), "status": state["status"]}
    buf = state["buf"]
    out = moe.run_layer(buf, state["x"], state["ids"], state["wts"], state["weights"])
    return {"out": out.view(torch.bfloat16), "status": buf.dev_status}


# -------------------------------------------------------------------- work

def _active_experts(case):
    """Expected experts with at least one token."""
    e, k, t = case["experts"], case["topk"], case["tokens"]
    p = [(r + 1) ** -case["zipf"] for r in range(e)]
    total = sum(p)
    return sum(1.0 - (1.0 - min(1.0, k * q / total)) ** t for q in p)


def work(case):
    t, h, i, e, k = case["tokens"], case["hidden"], case["inter"], case["experts"], case["topk"]
    if case["kind"] == "router":
        return {"bytes": 2.0 * t * h + 2.0 * e * h + 8.0 * t * k, "flops": 2.0 * t * h * e}
    experts = e if case["kind"] == "streamed" else _active_experts(case)
    per_expert = 3.0 * h * i * (1.0 + 4.0 / (BLOCK * BLOCK))
    return {"bytes": experts * per_expert + 4.0 * t * h + 8.0 * t * k, "flops": 6.0 * t * k * h * i}


def tolerance(case):
    if case["kind"] == "router":
        # Weights are 32-bit; a token whose groups tie within the rounding of
        # its logits may keep another group, and neighbours in the order swap.
        return {"rel": 3e-4, "max": 0.5, "differ": 5e-4}
    # bf16 output; a sum in another order moves some values of h across an
    # e4m3 rounding boundary before the down projection.
    return {"rel": 1e-2, "max": 0.1}


# ------------------------------------------------------------------- exact

def _quantize(x):
    """Rows quantized per 128 columns (fp32 in), as their dequantized values in 64 bits.

    Scale and quotient are the correctly rounded fp32 values (both through 64
    bits: bf16 activations hit many exact rounding midpoints, which a scale
    that is one unit off would move)."""
    b = x.to(torch.float64).view(x.shape[0], -1, BLOCK)
    s = (b.abs().amax(2, keepdim=True) / E4M3_MAX).to(torch.float32).to(torch.float64)
    q = torch.where(s > 0, b / s, torch.zeros_like(b)).to(torch.float32)
    q = q.clamp_(-E4M3_MAX, E4M3_MAX).to(torch.float8_e4m3fn)
    return (q.to(torch.float64) * s).view(x.shape)


def _dequant(codes, scales):
    s = scales.to(torch.float64).repeat_interleave(BLOCK, 0).repeat_interleave(BLOCK, 1)
    return codes.view(torch.float8_e4m3fn).to(torch.float64) * s


def _exact_layer(case, seed):
    wg, sg, wu, su, wd, sd = _weights(case, seed)
    x = _tokens(case, seed)
    ids, wts = _routing(case, seed)
    a16 = case["kind"] == "w8a16"
    xq = x.to(torch.float64) if a16 else _quantize(x.to(torch.float32))
    out = torch.zeros((case["tokens"], case["hidden"]), dtype=torch.float64, device="cuda")
    for e in range(case["experts"]):
        t, j = (ids == e).nonzero(as_tuple=True)
        if not len(t):
            continue
        a = xq[t]
        g = a @ _dequant(wg[e], sg[e]).t()
        u = a @ _dequant(wu[e], su[e]).t()
        hid = (g * torch.sigmoid(g) * u).to(torch.float32)
        hid = hid.to(torch.bfloat16).to(torch.float64) if a16 else _quantize(hid)
        out.index_add_(0, t, (hid @ _dequant(wd[e], sd[e]).t()) * wts[t, j].to(torch.float64)[:, None])
    return {"out": out, "status": None}


def exact(case, seed):
    if case["kind"] != "router":
        return _exact_layer(case, seed)
    x = _tokens(case, seed)
    w, bias = _gate(case, seed)
    k, n = case["topk"], case["groups"]
    s = torch.sigmoid(x.to(torch.float64) @ w.to(torch.float64).t())
    key = s if bias is None else s + bias.to(torch.float64)
    if n > 1:
        per = key.view(len(x), n, -1)
        kept = torch.topk(torch.topk(per, 2, dim=2).values.sum(2), case["kept"], dim=1).indices
        mask = torch.zeros((len(x), n), dtype=torch.bool, device="cuda").scatter_(1, kept, True)
        key = torch.where(mask[:, :, None], per, -torch.inf).view(key.shape)
    picked = s.gather(1, torch.topk(key, k, dim=1).indices)
    return {"ids": None, "weights": picked / picked.sum(1, keepdim=True) * 2.5}
