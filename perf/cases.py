"""Performance cases: the calls a serving program makes on this library, as plain dicts, with their inputs, the work they
cannot do without, the error they may show and their result in 64 bits.

Every case is one call of a public entry point on synthetic inputs of the shapes and distributions used throughout this
repository (weights N(0, 0.02^2) quantised per group, activations and cached keys / values N(0, 1), norm weights
1 + 0.1 N(0, 1)).  The keys of a case:

  op        "layer" (DeviceLayer / DeviceLayerQ3 / DeviceLayerF16.forward), "model" (DeviceModel.step), "attention"
            (relax_attention)
  hidden, heads, kv_heads, head_dim, ffn    the model's static sizes
  weights, group                            "q4" | "q3" | "f16", and the columns per scale of a 4-bit matrix
  prompt, past                              rows one sequence brings (0: no such sequence) on top of `past` cached tokens
  decodes, len_first, len_step              further sequences with one row each, lengths len_first + b * len_step
  layers, vocab                             of a "model" case
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2311_02103_amd import binding as rx
from paper_2311_02103_amd.runtime import DeviceLayer, DeviceLayerF16, DeviceLayerQ3, DeviceModel

EPS, ROPE_BASE = 1e-5, 10000.0

TINY = dict(hidden=256, heads=4, kv_heads=4, head_dim=64, ffn=688)
B7 = dict(hidden=4096, heads=32, kv_heads=32, head_dim=128, ffn=11008)
B13 = dict(hidden=5120, heads=40, kv_heads=40, head_dim=128, ffn=13824)
B70 = dict(hidden=8192, heads=64, kv_heads=8, head_dim=128, ffn=28672)


def _layer(shape, weights="q4", group=32, prompt=0, past=0, decodes=0, len_first=0, len_step=0):
    return dict(op="layer", weights=weights, group=group, prompt=prompt, past=past, decodes=decodes, len_first=len_first,
                len_step=len_step, **shape)


def _model(shape, layers, vocab, **seqs):
    case = _layer(shape, **seqs)
    case.update(op="model", layers=layers, vocab=vocab)
    return case


def _attention(shape, **seqs):
    case = _layer(shape, **seqs)
    case.update(op="attention")
    return case


def listed():
    return [
        # the smallest configuration: one greedy token of a toy model, nothing but launches and latency
        dict(name="tiny_decode", **_layer(TINY, decodes=1, len_first=53)),
        # interactive chat on one card: one token of one user, middle of a 4096-token context
        dict(name="7b_decode", **_layer(B7, decodes=1, len_first=2231)),
        # two layers with embedding and vocabulary projection: what a token costs besides its layers
        dict(name="7b_model_decode", **_model(B7, 2, 32000, decodes=1, len_first=385)),
        # a few users, or a few beams, on the middle model size with the coarser scales of most 4-bit deployments
        dict(name="13b_g128_decode_4", **_layer(B13, group=128, decodes=4, len_first=300, len_step=211)),
        # continuous batching at the largest batch that the batch sweep of the evaluation uses
        dict(name="7b_decode_64", **_layer(B7, decodes=64, len_first=128, len_step=13)),
        # long-context serving with grouped heads: sixteen users between 100 and 8000 tokens
        dict(name="70b_decode_16", **_layer(B70, decodes=16, len_first=100, len_step=526)),
        # a serving step that carries a chunk of one prompt beside the decode rows of other users
        dict(name="7b_mixed", **_layer(B7, prompt=300, past=1201, decodes=20, len_first=90, len_step=57)),
        # a prompt of odd length on the largest model
        dict(name="70b_prefill_511", **_layer(B70, prompt=511)),
        # a long prompt in one call
        dict(name="7b_prefill_2048", **_layer(B7, prompt=2048)),
        # a short prompt on 3-bit weights, the format of the small devices
        dict(name="7b_q3_prompt_17", **_layer(B7, weights="q3", prompt=17)),
        # a small batch on unquantised weights, the other half of the evaluation
        dict(name="7b_f16_decode_8", **_layer(B7, weights="f16", decodes=8, len_first=200, len_step=97)),
        # attention by itself over a long prompt with grouped heads
        dict(name="attention_4096", **_attention(dict(B7, kv_heads=8), prompt=4096)),
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.49)))))))


def _decode_lengths(rng, count, longest):
    first = _log(rng, 16, max(17, longest // 2))
    return dict(decodes=count, len_first=first, len_step=rng.randint(0, max(1, (longest - first) // max(1, count))))


def draw(rng):
    """One case of the ranges above: every family at every size between its smallest and its largest listed call."""
    family = rng.choice(["tiny", "decode", "decode", "decode", "mixed", "prefill", "prefill", "q3", "f16", "model", "attention"])
    if family == "tiny":
        n = _log(rng, 1, 37)
        return _layer(TINY, decodes=1, len_first=_log(rng, 1, 256)) if n == 1 else _layer(TINY, prompt=n, past=rng.choice([0, rng.randint(1, 200)]))
    if family == "decode":
        shape = rng.choice([B7, B13, B70])
        return _layer(shape, group=rng.choice([32, 32, 64, 128]), **_decode_lengths(rng, _log(rng, 1, 64), rng.choice([600, 2000, 4000])))
    if family == "mixed":
        return _layer(rng.choice([B7, B13]), group=rng.choice([32, 128]), prompt=_log(rng, 5, 400), past=rng.randint(0, 1500),
                      **_decode_lengths(rng, _log(rng, 1, 32), 1200))
    if family == "prefill":
        shape, most = rng.choice([(B7, 2048), (B13, 1024), (B70, 511)])
        return _layer(shape, group=rng.choice([32, 32, 64, 128]), prompt=_log(rng, 2, most), past=rng.choice([0, 0, rng.randint(1, 1500)]))
    if family in ("q3", "f16"):
        if rng.random() < 0.5:
            return _layer(B7, weights=family, **_decode_lengths(rng, _log(rng, 1, 24), 1500))
        return _layer(B7, weights=family, prompt=_log(rng, 2, 800), past=rng.choice([0, rng.randint(1, 500)]))
    if family == "model":
        return _model(B7, 2, 32000, **_decode_lengths(rng, _log(rng, 1, 24), 1000))
    heads, kv_heads, d = rng.choice([(32, 8, 128), (32, 32, 128), (64, 8, 128), (32, 8, 64)])
    shape = dict(hidden=heads * d, heads=heads, kv_heads=kv_heads, head_dim=d, ffn=4096)
    return _attention(shape, prompt=_log(rng, 40, 4096 if heads == 32 else 2500), past=rng.choice([0, rng.randint(1, 600)]))


# ---- shapes of a call -----------------------------------------------------------------------------------------------
def _seqs(c):
    """(q_lens, kv_lens) of the call: the prompt first, then the decode rows."""
    q, kv = [], []
    if c["prompt"]:
        q, kv = [c["prompt"]], [c["past"] + c["prompt"]]
    return q + [1] * c["decodes"], kv + [c["len_first"] + b * c["len_step"] for b in range(c["decodes"])]


def _mats(c):
    h, g, d = c["heads"], c["kv_heads"], c["head_dim"]
    return {"wqkv": ((h + 2 * g) * d, c["hidden"]), "wo": (c["hidden"], h * d), "wgu": (2 * c["ffn"], c["hidden"]),
            "wdown": (c["hidden"], c["ffn"])}


def _capacity(c):
    return (max(_seqs(c)[1]) + 63) // 64 * 64


def work(c):
    q, kv = _seqs(c)
    n, h, g, d, H = sum(q), c["heads"], c["kv_heads"], c["head_dim"], c["hidden"]
    pairs = sum(ql * (L - ql) + ql * (ql + 1) // 2 for ql, L in zip(q, kv))
    att_bytes, att_flops = sum(kv) * 2 * g * d * 2, 4 * pairs * h * d
    if c["op"] == "attention":
        return {"bytes": att_bytes + 2 * n * h * d * 2, "flops": att_flops}
    per = {"q4": 0.5 + 2.0 / c["group"], "q3": 0.375 + 2.0 / 32, "f16": 2.0}[c["weights"]]
    params = sum(m * k for m, k in _mats(c).values())
    by, fl = params * per + 2 * H * 2 + att_bytes + 2 * n * H * 2, 2 * n * params + att_flops
    if c["op"] == "model":
        by = by * c["layers"] + (c["vocab"] * H + len(q) * c["vocab"]) * 2
        fl = fl * c["layers"] + 2 * len(q) * c["vocab"] * H
    return {"bytes": by, "flops": fl}


def tolerance(c):
    # Activations, K / V and attention outputs are fp16 (2^-11 per rounding) between fp32 sums.  Seen against the 64-bit result:
    # attention 2.6e-4 (largest element 3.9e-3); a layer 2.0e-4 to 9.1e-4, on the 8192-wide model with a prompt, whose second half
    # adds sums of 28672 terms, 1.5e-3 (largest element 8.3e-3); two layers and the head 1.3e-3 (6.6e-3).  Four times that.
    if c["op"] == "attention":
        return {"rel": 1.1e-3, "max": 1.6e-2}
    return {"rel": 6e-3, "max": 3.3e-2}


# ---- inputs ---------------------------------------------------------------------------------------------------------
def _gen(seed, tensor):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed) * 1000003 + tensor)
    return g


def _normal(seed, tensor, shape, std=1.0, mean=0.0):
    t = torch.empty(shape, dtype=torch.float32, device="cuda").normal_(mean, std, generator=_gen(seed, tensor))
    return t.half()


def _quantised(seed, tensor, m, k, group, top):
    """(codes int32 [m, k] around zero, scales fp16 [m, ceil(k / group)]): round(w / s) with s = max|w| / top per group."""
    w = torch.empty((m, k), dtype=torch.float32, device="cuda").normal_(0.0, 0.02, generator=_gen(seed, tensor))
    groups = -(-k // group)
    w = torch.nn.functional.pad(w, (0, groups * group - k)).view(m, groups, group)
    s = (w.abs().amax(dim=2) / top).half()
    codes = torch.round(w / s.float().clamp_min(1e-8).unsqueeze(2)).clamp_(-top, top)
    return codes.view(m, groups * group)[:, :k].to(torch.int32), s


def _pack4(codes):
    m, k = codes.shape
    u = (codes + 8).view(m, k // 8, 8)
    word = torch.zeros((m, k // 8), dtype=torch.int32, device=codes.device)
    for j in range(8):
        word |= u[:, :, j] << (4 * j)
    return word


def _pack3(codes):
    """The canonical 3-bit layout: the 32 codes of a group end to end in three little-endian words."""
    m, k = codes.shape
    u = (codes + 4).view(m, k // 32, 32).to(torch.int64)
    words = torch.zeros((m, k // 32, 3), dtype=torch.int64, device=codes.device)
    for c in range(32):
        w, b = divmod(3 * c, 32)
        words[:, :, w] |= (u[:, :, c] << b) & 0xFFFFFFFF
        if b > 29:
            words[:, :, w + 1] |= u[:, :, c] >> (32 - b)
    return torch.where(words >= 2 ** 31, words - 2 ** 32, words).to(torch.int32).view(m, 3 * k // 32)


def _weights(c, seed, layer):
    """Per matrix its (codes, scales), or its fp16 values; and the two norm vectors."""
    out = {}
    for i, (name, (m, k)) in enumerate(_mats(c).items()):
        tensor = 100 + 16 * layer + i
        if c["weights"] == "f16":
            out[name] = _normal(seed, tensor, (m, k), std=0.02)
        else:
            out[name] = _quantised(seed, tensor, m, k, c["group"] if c["weights"] == "q4" else 32, 7 if c["weights"] == "q4" else 3)
    for i, name in enumerate(("norm_attn", "norm_ffn")):
        out[name] = _normal(seed, 110 + 16 * layer + i, (c["hidden"],), std=0.1, mean=1.0)
    return out


def _caches(c, seed, layer):
    shape = (len(_seqs(c)[0]), _capacity(c), c["kv_heads"], c["head_dim"])
    return _normal(seed, 50 + 2 * layer, shape), _normal(seed, 51 + 2 * layer, shape)


def _host_bits(t):
    return t.contiguous().view(torch.int16).cpu().numpy().view(np.uint16)


def _host_weights(c, w):
    """The host arrays a program would have read from its checkpoint."""
    host = {}
    for name in _mats(c):
        if c["weights"] == "f16":
            host[name] = _host_bits(w[name])
        else:
            codes, s = w[name]
            host[name + ".q"] = (_pack4 if c["weights"] == "q4" else _pack3)(codes).cpu().numpy().view(np.uint32)
            host[name + ".s"] = _host_bits(s)
    host["norm_attn"], host["norm_ffn"] = _host_bits(w["norm_attn"]), _host_bits(w["norm_ffn"])
    return host


def _sizes(c):
    q, kv = _seqs(c)
    return dict(hidden=c["hidden"], n_heads=c["heads"], n_kv_heads=c["kv_heads"], head_dim=c["head_dim"], ffn=c["ffn"],
                kv_capacity=_capacity(c), kv_slots=len(q), n_max=sum(q), rms_eps=EPS, rope_base=ROPE_BASE)


def _appended(c, cache):
    """Views of what the call writes into a cache: the rows of the prompt, and the row of every decode sequence."""
    q, kv = _seqs(c)
    views, first = [], 0
    token = cache.stride(1)
    if c["prompt"]:
        views.append(cache[0, c["past"]:c["past"] + c["prompt"]])
        first = 1
    if c["decodes"]:
        views.append(cache.as_strided((c["decodes"],) + tuple(cache.shape[2:]), (cache.stride(0) + c["len_step"] * token,) + cache.stride()[2:],
                                      cache.storage_offset() + first * cache.stride(0) + (c["len_first"] - 1) * token))
    return views


def _q(c, seed):
    return _normal(seed, 2, (sum(_seqs(c)[0]), c["heads"], c["head_dim"]))


def prepare(c, seed):
    q, kv = _seqs(c)
    state = {"case": c, "q_lens": q, "kv_lens": kv}
    if c["op"] == "attention":
        state["q"], (state["k"], state["v"]) = _q(c, seed), _caches(c, seed, 0)
        state["dims"] = rx.make_dims(c["hidden"], c["heads"], c["kv_heads"], c["head_dim"], c["ffn"], _capacity(c), len(q))
        rope = torch.empty(rx.relax_rope_table_bytes(state["dims"]) // 4, dtype=torch.float32, device="cuda")
        rx.check(rx.relax_rope_table_init(state["dims"], rope))
        state["cache"] = rx.KVCache(state["k"], state["v"], rope)
        state["ws_bytes"] = rx.relax_workspace_bytes(state["dims"], sum(q), max(kv), len(q))
        state["ws"] = torch.empty(state["ws_bytes"], dtype=torch.uint8, device="cuda")
        return state
    if c["op"] == "model":
        hosts = [_host_weights(c, _weights(c, seed, layer)) for layer in range(c["layers"])]
        emb, head, norm = _model_tensors(c, seed)
        m = DeviceModel(hosts, _host_bits(emb), _host_bits(norm), _host_bits(head), group=c["group"], **_sizes(c))
        for layer in range(c["layers"]):
            k, v = _caches(c, seed, layer)
            m.k[layer].copy_(k)
            m.v[layer].copy_(v)
        state["model"], state["ids"] = m, _ids(c, seed)
        state["appended"] = [_appended(c, t) for layer in range(c["layers"]) for t in (m.k[layer], m.v[layer])]
        return state
    kind = {"q4": DeviceLayer, "q3": DeviceLayerQ3, "f16": DeviceLayerF16}[c["weights"]]
    more = {"group": c["group"]} if c["weights"] == "q4" else {}
    layer = kind(_host_weights(c, _weights(c, seed, 0)), **_sizes(c), **more)
    k, v = _caches(c, seed, 0)
    layer.k.copy_(k)
    layer.v.copy_(v)
    state["layer"], state["x"] = layer, _normal(seed, 1, (sum(q), c["hidden"]))
    state["appended"] = [_appended(c, layer.k), _appended(c, layer.v)]
    return state


def _model_tensors(c, seed):
    return (_normal(seed, 20, (c["vocab"], c["hidden"]), std=0.02), _normal(seed, 21, (c["vocab"], c["hidden"]), std=0.02),
            _normal(seed, 22, (c["hidden"],), std=0.1, mean=1.0))


def _ids(c, seed):
    return torch.randint(0, c["vocab"], (sum(_seqs(c)[0]),), dtype=torch.int32, device="cuda", generator=_gen(seed, 3))


def run(state):
    if "layer" in state:
        out = state["layer"].forward(state["x"], state["q_lens"], state["kv_lens"])
        return [out, state["appended"]]
    if "model" in state:
        logits, _ = state["model"].step(state["ids"], state["q_lens"], state["kv_lens"])
        return [logits, state["appended"]]
    out = torch.empty_like(state["q"])
    seqs = rx.Seqs(state["q_lens"], state["kv_lens"])
    rx.check(rx.relax_attention(state["q"], state["cache"], seqs, state["dims"], out, out.shape[0], state["ws"], state["ws_bytes"]),
             "relax_attention")
    return [out]


# ---- the same in 64 bits, plain torch -------------------------------------------------------------------------------
def _times(x, c, w):
    """x [n, k] times the transposed matrix, in slabs of rows."""
    if c["weights"] == "f16":
        return x @ w.double().t()
    codes, s = w
    group = c["group"] if c["weights"] == "q4" else 32
    parts = []
    for r in range(0, codes.shape[0], 4096):
        scale = s[r:r + 4096].double().repeat_interleave(group, dim=1)[:, :codes.shape[1]]
        parts.append(x @ (codes[r:r + 4096].double() * scale).t())
    return torch.cat(parts, dim=1)


def _rms(x, w):
    return x * torch.rsqrt((x * x).mean(dim=1, keepdim=True) + EPS) * w.double()


def _rope(x, pos):
    """Half-split rotary embedding of x [n, heads, d] at positions pos [n]."""
    half = x.shape[2] // 2
    angle = pos.double()[:, None] * ROPE_BASE ** (-torch.arange(half, device=x.device, dtype=torch.float64) / half)
    cos, sin = angle.cos()[:, None], angle.sin()[:, None]
    a, b = x[:, :, :half], x[:, :, half:]
    return torch.cat([a * cos - b * sin, a * sin + b * cos], dim=2)


def _attend(c, q, k, v):
    """q [n, h, d]; k, v: caches [slots, capacity, g, d] in any precision that hold this call's rows too."""
    out, row, rep = torch.empty_like(q), 0, c["heads"] // c["kv_heads"]
    for slot, (ql, L) in enumerate(zip(*_seqs(c))):
        mask = torch.arange(L, device=q.device)[None] > torch.arange(L - ql, L, device=q.device)[:, None]
        for g in range(c["kv_heads"]):
            kg, vg = k[slot, :L, g].double(), v[slot, :L, g].double()
            for j in range(g * rep, (g + 1) * rep):
                s = (q[row:row + ql, j] @ kg.t() / math.sqrt(c["head_dim"])).masked_fill(mask, -math.inf)
                out[row:row + ql, j] = torch.softmax(s, dim=1) @ vg
        row += ql
    return out


def _exact_layer(c, w, x, k, v):
    """The layer's output; the call's rows are put into k and v (float64 caches)."""
    h, g, d = c["heads"], c["kv_heads"], c["head_dim"]
    q_lens, kv_lens = _seqs(c)
    pos = torch.cat([torch.arange(L - ql, L, device=x.device) for ql, L in zip(q_lens, kv_lens)])
    slot = torch.cat([torch.full((ql,), b, device=x.device) for b, ql in enumerate(q_lens)])
    qkv = _times(_rms(x, w["norm_attn"]), c, w["wqkv"])
    q = _rope(qkv[:, :h * d].view(-1, h, d), pos)
    k[slot, pos] = _rope(qkv[:, h * d:(h + g) * d].reshape(-1, g, d), pos)
    v[slot, pos] = qkv[:, (h + g) * d:].reshape(-1, g, d)
    x = x + _times(_attend(c, q, k, v).reshape(-1, h * d), c, w["wo"])
    gate, up = _times(_rms(x, w["norm_ffn"]), c, w["wgu"]).chunk(2, dim=1)
    return x + _times(torch.nn.functional.silu(gate) * up, c, w["wdown"])


def exact(c, seed):
    if c["op"] == "attention":
        return [_attend(c, _q(c, seed).double(), *_caches(c, seed, 0))]
    x, appended = None, []
    if c["op"] == "model":
        emb, head, norm = _model_tensors(c, seed)
        x = emb[_ids(c, seed).long()].double()
    else:
        x = _normal(seed, 1, (sum(_seqs(c)[0]), c["hidden"])).double()
    for layer in range(c.get("layers", 1)):
        k, v = (t.double() for t in _caches(c, seed, layer))
        x = _exact_layer(c, _weights(c, seed, layer), x, k, v)
        appended += [_appended(c, k), _appended(c, v)]
    if c["op"] == "layer":
        return [x, appended]
    last = torch.tensor(_seqs(c)[0], device=x.device).cumsum(0) - 1
    return [_rms(x[last], norm) @ head.double().t(), appended]
