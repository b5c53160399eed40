"""Performance cases of the W4A16 routed-expert layer and the decoder around it.

Every case is a call, or one model step of calls, that a program using this
framework makes through its public Python entry points: the layer call at
decode, batched-decode and prefill sizes, the layer behind a slot cache, the
offline quantization, and the decoder's prompt and decode step.  The main
shape is the OLMoE-shaped layer of this repository's benchmark (d_model 2048,
d_ff 1024, 64 experts, top-8, 16 layers); the small shapes are the tests'.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2608_15383_amd import api
from paper_2608_15383_amd.inputs import spread_logits, zipf_gumbel_logits

OLMOE = dict(d=2048, f=1024, experts=64, k=8)
GROUP = 128
HEADS, HEAD_DIM, VOCAB, MAX_POS = 16, 128, 50304, 512
ROPE_BASE, RMS_EPS = 10000.0, 1e-5


def _layer(name, tokens, layers=1, routing="router", renorm=True, shape=OLMOE):
    return dict(name=name, kind="layer", tokens=tokens, layers=layers, routing=routing,
                renorm=renorm, **shape)


def listed():
    return [
        # One decoded token through the model's 16 expert layers, each with its
        # own bank, so the weights come from memory as in a running model.
        _layer("decode_1", 1, layers=16),
        # Four sequences decoded together.
        _layer("decode_4", 4, layers=16),
        # A small decode batch: nearly every expert active, one or two rows each.
        _layer("batch_16", 16, layers=4),
        # A decode batch of odd size, weights not renormalized (the option that
        # keeps the softmax over all experts).
        _layer("batch_113", 113, layers=4, renorm=False),
        # A ragged prompt with skewed expert popularity (Zipf 1.1).
        _layer("prefill_777_zipf", 777, routing="zipf"),
        # The benchmark's prefill.
        _layer("prefill_2048", 2048),
        # The smallest layer of the tests: launches and latency only.
        _layer("tiny_16", 16, shape=dict(d=256, f=128, experts=8, k=2)),
        # Sizes that no tile divides: 5 and 3 groups, 12 experts, top-3.
        _layer("ragged_301", 301, shape=dict(d=640, f=384, experts=12, k=3)),
        # 16 tokens on 56 experts through 16 slots over a pinned host bank.
        dict(name="slots_16", kind="slots", tokens=16, distinct=56, capacity=16, overlap=False,
             **OLMOE),
        # Offline conversion of one layer's experts.
        dict(name="quantize_64", kind="quantize", n=64, **OLMOE),
        # The decoder's prompt (time to first token) and a decode step in the
        # middle of a request.
        dict(name="decoder_prompt_128", kind="decoder", tokens=128, pos0=0, layers=16, **OLMOE),
        dict(name="decoder_step", kind="decoder", tokens=1, pos0=301, layers=16, **OLMOE),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["decode", "batch", "prefill", "prefill", "small", "small", "slots",
                       "quantize", "prompt", "step"])
    if kind == "decode":
        return _unnamed(_layer("", rng.randint(1, 4), layers=rng.randint(8, 16),
                               renorm=rng.random() < 0.5))
    if kind == "batch":
        return _unnamed(_layer("", _log_int(rng, 5, 200), layers=rng.randint(2, 4),
                               routing=rng.choice(["router", "zipf"]),
                               renorm=rng.random() < 0.5))
    if kind == "prefill":
        return _unnamed(_layer("", _log_int(rng, 200, 2048),
                               routing=rng.choice(["router", "zipf"]),
                               renorm=rng.random() < 0.5))
    if kind == "small":
        experts = rng.randint(4, 96)
        shape = dict(d=128 * rng.randint(1, 8), f=128 * rng.randint(1, 8), experts=experts,
                     k=rng.randint(1, min(8, experts)))
        return _unnamed(_layer("", _log_int(rng, 1, 512), shape=shape,
                               routing=rng.choice(["router", "zipf"]),
                               renorm=rng.random() < 0.5))
    if kind == "slots":
        return dict(kind="slots", tokens=rng.randint(7, 16), distinct=rng.randint(24, 56),
                    capacity=rng.randint(12, 24), overlap=rng.random() < 0.5, **OLMOE)
    if kind == "quantize":
        shape = dict(OLMOE) if rng.random() < 0.5 else dict(
            d=128 * rng.randint(2, 16), f=128 * rng.randint(1, 8), experts=64, k=8)
        return dict(kind="quantize", n=_log_int(rng, 4, 64), **shape)
    if kind == "prompt":
        return dict(kind="decoder", tokens=_log_int(rng, 12, 128), pos0=0, layers=16, **OLMOE)
    return dict(kind="decoder", tokens=rng.randint(1, 4), pos0=_log_int(rng, 16, 500), layers=16,
                **OLMOE)


def _unnamed(case):
    case.pop("name")
    return case


# ---------------------------------------------------------------- inputs
def _gen(seed, tag):
    return torch.Generator(device="cuda").manual_seed((seed * 1_000_003 + 7919 * tag) % (1 << 62))


def _normal(g, shape, scale, shift=0.0):
    x = torch.randn(shape, dtype=torch.float32, device="cuda", generator=g)
    return (x * scale + shift).to(torch.bfloat16)


def _expert_weights(case, seed, layer, n):
    """bf16 gate, up [n][f][d] and down [n][d][f] of one layer, ~N(0, 0.02)."""
    g = _gen(seed, 100 + layer)
    d, f = case["d"], case["f"]
    return _normal(g, (n, f, d), 0.02), _normal(g, (n, f, d), 0.02), _normal(g, (n, d, f), 0.02)


def _token_rows(case, seed, layer):
    return _normal(_gen(seed, 300 + layer), (case["tokens"], case["d"]), 1.0)


def _router(case, seed, layer):
    return _normal(_gen(seed, 500 + layer), (case["experts"], case["d"]), 0.02)


def _given_logits(case, seed, layer):
    """Routing logits handed to the call (None: the call's own router)."""
    if case["kind"] == "slots":
        z = spread_logits(case["tokens"], case["experts"], case["k"], case["distinct"], seed)
    elif case.get("routing") == "zipf":
        rng = np.random.default_rng([seed, layer])
        z = zipf_gumbel_logits(case["tokens"], case["experts"], 1.1,
                               rng.permutation(case["experts"]), rng)
    else:
        return None
    return torch.from_numpy(z).to("cuda")


def _dims(case):
    return api.dims(case["d"], case["f"], case["experts"], case["k"])


def _quantized_bank(case, dm, seed, layer):
    n = case["experts"]
    wg, wu, wd = _expert_weights(case, seed, layer, n)
    bank = torch.empty(n * api.expert_record_bytes(dm), dtype=torch.uint8, device="cuda")
    api.quantize_experts(dm, wg, wu, wd, bank)
    return bank


def _resident_cache(case, dm, seed, layer):
    bank = _quantized_bank(case, dm, seed, layer)
    cache = api.Cache(dm, case["experts"], slot_bank=bank)
    cache.preload_all()
    return cache


def _decoder_weights(case, seed):
    d, n = case["d"], case["layers"]
    g = _gen(seed, 1)
    w = dict(embed=_normal(g, (VOCAB, d), 1.0), lm_head=_normal(g, (VOCAB, d), 0.02),
             final_norm=_normal(g, (d,), 0.1, 1.0))
    w["attn_norm"] = [_normal(g, (d,), 0.1, 1.0) for _ in range(n)]
    w["wqkv"] = [_normal(g, (3 * d, d), 0.02) for _ in range(n)]
    w["wo"] = [_normal(g, (d, d), 0.02) for _ in range(n)]
    w["moe_norm"] = [_normal(g, (d,), 0.1, 1.0) for _ in range(n)]
    w["w_router"] = [_router(case, seed, l) for l in range(n)]
    return w


def _decoder_tokens(case, seed):
    return torch.randint(0, VOCAB, (case["tokens"],), dtype=torch.int32, device="cuda",
                         generator=_gen(seed, 2))


def _decoder_history(case, seed):
    """KV cache [layer][k, v][position][d] with pos0 earlier positions filled."""
    kv = torch.zeros((case["layers"], 2, MAX_POS, case["d"]), dtype=torch.bfloat16, device="cuda")
    if case["pos0"]:
        kv[:, :, :case["pos0"]] = _normal(
            _gen(seed, 3), (case["layers"], 2, case["pos0"], case["d"]), 0.9)
    return kv


def prepare(case, seed):
    dm = _dims(case)
    kind = case["kind"]
    if kind == "quantize":
        wg, wu, wd = _expert_weights(case, seed, 0, case["n"])
        rec = torch.empty(case["n"] * api.expert_record_bytes(dm), dtype=torch.uint8, device="cuda")
        return dict(kind=kind, dm=dm, weights=(wg, wu, wd), records=rec)
    if kind == "decoder":
        dd = api.decoder_dims(case["layers"], HEADS, HEAD_DIM, VOCAB, MAX_POS, dm, ROPE_BASE, RMS_EPS)
        caches = [_resident_cache(case, dm, seed, l) for l in range(case["layers"])]
        kv = _decoder_history(case, seed)
        weights = _decoder_weights(case, seed)
        return dict(kind=kind, pos0=case["pos0"], kv=kv, caches=caches, weights=weights,
                    decoder=api.Decoder(dd, weights, caches, kv),
                    tokens=_decoder_tokens(case, seed),
                    logits=torch.empty(VOCAB, dtype=torch.float32, device="cuda"),
                    next_token=torch.empty(1, dtype=torch.int32, device="cuda"),
                    workspace=torch.empty(api.decoder_workspace_bytes(dd, case["tokens"]),
                                          dtype=torch.uint8, device="cuda"))
    layers = []
    for l in range(case.get("layers", 1)):
        if kind == "slots":
            bank = _quantized_bank(case, dm, seed, l)
            host = torch.empty(bank.numel(), dtype=torch.uint8, pin_memory=True)
            host.copy_(bank)
            slots = torch.zeros(case["capacity"] * api.expert_record_bytes(dm), dtype=torch.uint8,
                                device="cuda")
            cache = api.Cache(dm, case["capacity"], slot_bank=slots, host_bank=host)
            cache.set_wave_overlap(case["overlap"])
        else:
            cache = _resident_cache(case, dm, seed, l)
        h = _token_rows(case, seed, l)
        layers.append((cache, h, _router(case, seed, l), torch.empty_like(h),
                       _given_logits(case, seed, l)))
    ws = torch.empty(api.workspace_bytes(dm, case["tokens"]), dtype=torch.uint8, device="cuda")
    return dict(kind=kind, layers=layers, workspace=ws, renorm=case.get("renorm", True))


def run(state):
    if state["kind"] == "quantize":
        api.quantize_experts(state["dm"], *state["weights"], state["records"])
        return state["records"]
    if state["kind"] == "decoder":
        state["decoder"].forward(state["tokens"], state["pos0"], state["logits"],
                                 state["next_token"], state["workspace"])
        return dict(logits=state["logits"], kv=state["kv"])
    for cache, h, w_router, y, logits in state["layers"]:
        api.moe_forward(cache, h, w_router, y, state["workspace"], logits_override=logits,
                        renormalize=state["renorm"])
    return [y for _, _, _, y, _ in state["layers"]]


# ---------------------------------------------------------------- work
def _record_bytes(case):
    return 3 * case["f"] * case["d"] // 2 + 3 * case["f"] * case["d"] // 64


def _distinct(case):
    """Expected number of distinct experts of a call (uniform routing)."""
    if "distinct" in case:
        return min(case["distinct"], case["tokens"] * case["k"])
    e = case["experts"]
    return e * (1.0 - (1.0 - case["k"] / e) ** case["tokens"])


def _layer_work(case):
    t, d, f, e, k = (case[x] for x in ("tokens", "d", "f", "experts", "k"))
    given = case["kind"] == "slots" or case.get("routing") == "zipf"
    routing = 4 * t * e if given else 2 * e * d
    return (int(_distinct(case) * _record_bytes(case)) + routing + 4 * t * d,
            6 * t * k * d * f + (0 if given else 2 * t * e * d))


def work(case):
    d = case["d"]
    if case["kind"] == "quantize":
        return dict(bytes=case["n"] * (6 * case["f"] * d + _record_bytes(case)),
                    flops=case["n"] * 6 * case["f"] * d)
    nbytes, flops = _layer_work(case)
    n = case.get("layers", 1)
    if case["kind"] != "decoder":
        return dict(bytes=n * nbytes, flops=n * flops)
    t, p = case["tokens"], case["pos0"]
    keys = sum(p + i + 1 for i in range(t))
    nbytes += 2 * 4 * d * d + 4 * d * (p + t) + 4 * d * t
    flops += 2 * t * 4 * d * d + 4 * keys * d
    return dict(bytes=n * nbytes + 2 * VOCAB * d + 4 * VOCAB + 2 * t * d,
                flops=n * flops + 2 * VOCAB * d)


def tolerance(case):
    if case["kind"] == "quantize":
        return "exact"
    if case["kind"] == "decoder":
        # 16 layers in bf16: 0.01 .. 0.07 (logits) and 0.002 .. 0.02 (cache) from
        # the 64-bit result, the larger ones where rounding moved a token's last
        # expert.
        return {"rel": 0.15}
    # bf16 activations and outputs: 2.3e-3 .. 2.9e-3 from the 64-bit result.
    return {"rel": 1.2e-2}


# ---------------------------------------------------------------- 64-bit results
def _quantize(w):
    """Codes (float32 integers) and fp16 scales of w [N][K], per 128 inputs."""
    n, k = w.shape
    g = w.float().reshape(n, k // GROUP, GROUP)
    # A tensor divisor: torch multiplies by the reciprocal of a number.
    s32 = g.abs().amax(dim=2, keepdim=True) / torch.full((), 7.0, device=w.device).expand(1, 1, 1)
    s16 = s32.half()
    zero = s16.float() == 0
    q = torch.where(zero, torch.zeros_like(g), torch.round(g / s32).clamp(-8, 7))
    return q, torch.where(zero, torch.zeros_like(s16), s16)


def _dequantized(w):
    q, s = _quantize(w)
    return (q.double() * s.double()).reshape(w.shape)


def _packed(w):
    """Packed code tiles and scale lines of one matrix [N][K] as byte tensors."""
    n, k = w.shape
    q, s = _quantize(w)
    u = (q.reshape(n, k) + 8).to(torch.int32)
    # [row block][row][group][dword][quarter][pair][parity]
    u = u.reshape(n // 16, 16, k // GROUP, 4, 4, 4, 2).permute(0, 2, 4, 1, 3, 5, 6)
    shift = torch.tensor([[0, 16], [4, 20], [8, 24], [12, 28]], device=w.device)
    words = (u.long() << shift).sum(dim=(-1, -2))
    codes = torch.stack([(words >> (8 * b)) & 255 for b in range(4)], dim=-1).to(torch.uint8)
    scales = s.reshape(n // 64, 4, 16, k // GROUP).permute(0, 3, 2, 1).contiguous()
    return codes.reshape(-1), scales.reshape(-1).view(torch.uint8)


def _exact_records(case, seed):
    wg, wu, wd = _expert_weights(case, seed, 0, case["n"])
    d, f = case["d"], case["f"]
    out = []
    for e in range(case["n"]):
        w13 = torch.stack([wg[e].reshape(f // 16, 16, d), wu[e].reshape(f // 16, 16, d)], dim=1)
        for w in (w13.reshape(2 * f, d), wd[e]):
            out.extend(_packed(w))
    return torch.cat(out)


def _route(logits, k, renorm):
    z = logits.double()
    ids = torch.topk(z, k, dim=1).indices
    p = torch.softmax(z, dim=1).gather(1, ids)
    return ids, p / p.sum(dim=1, keepdim=True) if renorm else p


def _exact_moe(case, seed, layer, h, w_router, logits, renorm):
    """Eq. 1-2 in fp64 on the dequantized weights; h is fp64 [T][d]."""
    if logits is None:
        logits = (h @ w_router.double().T).float()
    ids, p = _route(logits, case["k"], renorm)
    wg, wu, wd = _expert_weights(case, seed, layer, case["experts"])
    y = torch.zeros_like(h)
    for e in range(case["experts"]):
        t, j = torch.nonzero(ids == e, as_tuple=True)
        if t.numel() == 0:
            continue
        x = h[t]
        gate = x @ _dequantized(wg[e]).T
        act = gate * torch.sigmoid(gate) * (x @ _dequantized(wu[e]).T)
        y.index_add_(0, t, p[t, j, None] * (act @ _dequantized(wd[e]).T))
    return y


def _rms(x, g):
    return x / torch.sqrt((x * x).mean(dim=-1, keepdim=True) + RMS_EPS) * g.double()


def _rope(x, pos):
    half = HEAD_DIM // 2
    inv = ROPE_BASE ** (-2.0 * torch.arange(half, dtype=torch.float64, device="cuda") / HEAD_DIM)
    ang = pos[:, None, None] * inv
    a, b = x[..., :half], x[..., half:]
    c, s = torch.cos(ang), torch.sin(ang)
    return torch.cat([a * c - b * s, b * c + a * s], dim=-1)


def _exact_decoder(case, seed):
    w = _decoder_weights(case, seed)
    kv = _decoder_history(case, seed).double()
    t, p0, d = case["tokens"], case["pos0"], case["d"]
    pos = torch.arange(p0, p0 + t, dtype=torch.float64, device="cuda")
    visible = torch.arange(p0 + t, device="cuda")[None, :] <= pos[:, None]
    x = w["embed"][_decoder_tokens(case, seed).long()].double()
    for l in range(case["layers"]):
        qkv = _rms(x, w["attn_norm"][l]) @ w["wqkv"][l].double().T
        q, k, v = (a.reshape(t, HEADS, HEAD_DIM) for a in qkv.split(d, dim=1))
        kv[l, 0, p0:p0 + t] = _rope(k, pos).reshape(t, d)
        kv[l, 1, p0:p0 + t] = v.reshape(t, d)
        q = _rope(q, pos).transpose(0, 1).contiguous()
        keys, vals = (kv[l, i, :p0 + t].reshape(-1, HEADS, HEAD_DIM).transpose(0, 1).contiguous()
                      for i in (0, 1))
        s = (q @ keys.transpose(1, 2).contiguous()) / math.sqrt(HEAD_DIM)
        s = torch.softmax(s.masked_fill(~visible, -math.inf), dim=-1)
        x = x + (s @ vals).transpose(0, 1).reshape(t, d) @ w["wo"][l].double().T
        n = _rms(x, w["moe_norm"][l])
        x = x + _exact_moe(case, seed, l, n, w["w_router"][l], None, True)
    logits = w["lm_head"].double() @ _rms(x[-1], w["final_norm"])
    return dict(logits=logits, kv=kv)


def exact(case, seed):
    if case["kind"] == "quantize":
        return _exact_records(case, seed)
    if case["kind"] == "decoder":
        return _exact_decoder(case, seed)
    return [_exact_moe(case, seed, l, _token_rows(case, seed, l).double(), _router(case, seed, l),
                       _given_logits(case, seed, l), case.get("renorm", True))
            for l in range(case.get("layers", 1))]
