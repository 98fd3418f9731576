"""Workloads by which the library's speed is measured, through its public entry points.

Each case is one call that a program built on this library makes: a decode token-layer (one token,
or several in one pair of launches), a dense FFN, a prefill layer, weight quantisation at load
time, or batch routing.  Shapes are those of the synthetic workloads (DeepSeek-V2-Lite-shaped and
Qwen1.5-MoE-shaped layers, the tiny fp32 layer) and generic ones of the same kinds.

`exact` recomputes every output with plain torch in 64 bits from the same dense weights; only the
quantiser keeps its fp32 arithmetic there, because that arithmetic defines the codes.
"""
from __future__ import annotations

import math

import torch

from paper_2512_12990_amd import binding as B

DEV = "cuda:0"
NESTS = {"8/4": (8, 4), "6/3": (6, 3), "4/2": (4, 2)}
DT = {"f32": torch.float32, "bf16": torch.bfloat16}


# ------------------------------------------------------------------------------------------- cases
def _layer(**kw):
    """A layer's shape and options; what a case leaves out is the plain form."""
    c = dict(d_model=2048, n_experts=64, d_ff=1408, top_k=6, group=128, n_shared=0, shared_d_ff=0, shared_gate=False,
             act="bf16", nest="8/4", symmetric=False, matvec=False, residual=False, norm_topk=False, tokens=1)
    c.update(kw)
    return c


def listed():
    dsv2 = dict(n_experts=64, d_ff=1408, top_k=6, n_shared=2, shared_d_ff=1408)
    qwen = dict(n_experts=60, d_ff=1408, top_k=4)
    qwen_sh = dict(qwen, n_shared=1, shared_d_ff=5632, shared_gate=True)
    return [
        # the smallest call: a tiny fp32 layer, three launches and nothing else
        _layer(name="decode-tiny-f32", kind="decode", d_model=256, n_experts=8, d_ff=128, top_k=2, group=64, act="f32", matvec=True),
        # one token through a DeepSeek-V2-Lite-shaped layer, cache mask and routing bias from a slice cache
        _layer(name="decode-dsv2", kind="decode", **dsv2),
        # one token of a Qwen1.5-MoE-shaped stack: router mat-vec, gated shared expert, residual
        _layer(name="decode-qwen-router", kind="decode", matvec=True, residual=True, **qwen_sh),
        # the dense first layer of a DeepSeek-V2-Lite-shaped stack (ragged last group: 10944 = 85*128 + 64)
        _layer(name="ffn-dense", kind="ffn", n_experts=0, d_ff=0, top_k=0, n_shared=1, shared_d_ff=10944, residual=True),
        # a short speculative draft in one call, 6/3 nest with the paper's groups of 32
        _layer(name="decode-multi-5-nest63", kind="decode", tokens=5, nest="6/3", **dict(dsv2, group=32)),
        # the widest multi-token step
        _layer(name="decode-multi-16", kind="decode", tokens=16, **dsv2),
        # a short, odd-sized prompt with plain shared experts
        _layer(name="prefill-dsv2-173", kind="prefill", tokens=173, matvec=True, **dsv2),
        # the warm-up prefill: 2048 tokens through a Qwen-shaped layer's routed experts
        _layer(name="prefill-qwen-2048", kind="prefill", tokens=2048, matvec=True, **qwen),
        # a long prompt through the whole Qwen-shaped layer
        _layer(name="prefill-qwen-shared-4096", kind="prefill", tokens=4096, matvec=True, residual=True, **qwen_sh),
        # model loading: bf16 expert weights into the 8/4 store
        _layer(name="quantize-bf16-84", kind="quantize", n_experts=8),
        # model loading: fp32 weights, 6/3 nest, groups of 32
        _layer(name="quantize-f32-63-g32", kind="quantize", n_experts=3, act="f32", nest="6/3", group=32),
        # routing decisions of a token batch alone, cache-aware, normalised weights
        _layer(name="route-1000", kind="route", tokens=1000, matvec=True, norm_topk=True),
    ]


def draw(rng):
    kind = rng.choice(["decode", "decode", "multi", "ffn", "prefill", "prefill", "quantize", "route"])
    log = lambda lo, hi: int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    act = "bf16" if kind in ("prefill", "multi") or rng.random() < 0.75 else "f32"
    c = _layer(kind="decode" if kind == "multi" else kind, act=act, nest=rng.choice(["8/4", "8/4", "6/3", "4/2"]),
               symmetric=rng.random() < 0.2, group=rng.choice([32, 64, 128, 128]), residual=rng.random() < 0.5,
               norm_topk=rng.random() < 0.3)
    c["d_model"] = 64 * log(4, 40)
    c["d_ff"] = 64 * log(2, 32)
    c["n_experts"] = log(8, 96)
    c["top_k"] = rng.randint(1, 8)
    c["matvec"] = kind != "multi" and rng.random() < 0.5
    if kind in ("decode", "multi", "prefill") and rng.random() < 0.5:
        c["n_shared"] = rng.randint(1, 2)
        c["shared_d_ff"] = 64 * log(2, 60)
        c["shared_gate"] = rng.random() < 0.5
    if kind == "multi":
        c["tokens"] = rng.randint(2, 16)
    elif kind == "prefill":
        c["tokens"] = log(20, 3000)
    elif kind == "route":
        c["tokens"] = log(20, 4000)
        c["matvec"] = True
    elif kind == "ffn":
        c.update(matvec=False)
        if rng.random() < 0.5:
            c.update(n_experts=0, d_ff=0, top_k=0, n_shared=1, shared_d_ff=64 * log(8, 170))
    elif kind == "quantize":
        c.update(n_experts=rng.randint(1, 6), matvec=False)
    return c


# ------------------------------------------------------------------------------------------ inputs
def _gen(seed, tag):
    g = torch.Generator(device=DEV)
    g.manual_seed((seed * 1000003 + tag * 7919 + 17) & 0x7FFFFFFF)
    return g


def _dense(case, seed, e, shared=False):
    """Dense weights of expert e, ~ N(0, 0.02^2), in the layer's dtype."""
    d, f = case["d_model"], case["shared_d_ff"] if shared else case["d_ff"]
    g = _gen(seed, 100 + e + (1000 if shared else 0))
    return tuple((torch.randn(s, generator=g, device=DEV) * 0.02).to(DT[case["act"]]) for s in ((f, d), (f, d), (d, f)))


def _inputs(case, seed):
    """Activations (a few channels carry outliers, as hidden states do), router inputs, cache state."""
    T, d, E, k = case["tokens"], case["d_model"], case["n_experts"], case["top_k"]
    s = {}
    x = torch.randn((T, d), generator=_gen(seed, 1), device=DEV)
    x[:, torch.randperm(d, generator=_gen(seed, 2), device=DEV)[: max(1, d // 256)]] *= 10.0
    s["x"] = x.to(DT[case["act"]])
    if E:
        s["logits"] = None if case["matvec"] else torch.randn((T, E), generator=_gen(seed, 3), device=DEV)
        s["w_router"] = torch.randn((E, d), generator=_gen(seed, 4), device=DEV) * 0.02 if case["matvec"] else None
        # half of the experts are resident (routing bias 1), half of those with both slices
        perm = torch.randperm(E, generator=_gen(seed, 5), device=DEV)
        mask = torch.zeros(E, dtype=torch.uint8, device=DEV)
        mask[perm[: E // 2]] = 1
        mask[perm[: E // 4]] = 3
        s["mask"], s["bias"] = mask, (mask > 0).float()
    s["gate"] = (torch.randn(d, generator=_gen(seed, 6), device=DEV) * 0.02).to(DT[case["act"]]) if case["shared_gate"] else None
    if case["kind"] == "ffn" and E:      # the routing decision is in hand
        s["idx"] = torch.randperm(E, generator=_gen(seed, 7), device=DEV)[:k].to(torch.int32)
        s["w"] = torch.rand(k, generator=_gen(seed, 8), device=DEV) * 0.3
    return s


def _bank(ctx, case, seed, shared=False):
    n, f = (case["n_shared"], case["shared_d_ff"]) if shared else (case["n_experts"], case["d_ff"])
    if n == 0:
        return None
    hi, lo = NESTS[case["nest"]]
    bank = B.Bank(ctx, n, case["d_model"], f, case["group"], case["act"], case["act"], hi, lo, case["symmetric"])
    bank.store.zero_()
    if case["kind"] != "quantize":
        for e in range(n):
            B.smoe_quantize_slice(ctx, bank, e, *(w[None] for w in _dense(case, seed, e, shared)))
    return bank


def prepare(case, seed):
    need = B.smoe_workspace_bytes(min(case["tokens"], 16), case["top_k"], case["d_ff"], case["n_shared"], case["shared_d_ff"])
    ctx = B.Ctx(0, workspace_bytes=need)
    s = {"case": case, "ctx": ctx}
    if case["kind"] == "quantize":
        s["bank"] = _bank(ctx, case, seed)
        ws = [_dense(case, seed, e) for e in range(case["n_experts"])]
        s["weights"] = [torch.stack([w[i] for w in ws]) for i in range(3)]
        return s
    s.update(_inputs(case, seed))
    if case["kind"] != "route":
        s["routed"], s["shared"] = _bank(ctx, case, seed), _bank(ctx, case, seed, shared=True)
    T, k = case["tokens"], case["top_k"]
    if case["kind"] in ("decode", "ffn"):
        s["y"] = torch.empty_like(s["x"])
        s["prec"] = torch.zeros((T, k), dtype=torch.uint8, device=DEV) if k else None
    if case["kind"] == "decode":
        s["idx"] = torch.empty((T, k), dtype=torch.int32, device=DEV)
        s["w"] = torch.empty((T, k), dtype=torch.float32, device=DEV)
    if case["kind"] == "prefill":
        n = B.smoe_prefill_bytes(T, case["n_experts"], k, case["d_model"], case["d_ff"], case["shared_d_ff"])
        s["scratch"] = torch.empty(n, dtype=torch.uint8, device=DEV)
    return s


# --------------------------------------------------------------------------------------- one pass
def run(s):
    c, ctx = s["case"], s["ctx"]
    kind = c["kind"]
    if kind == "quantize":
        B.smoe_quantize_slice(ctx, s["bank"], 0, *s["weights"])
        return {"store": s["bank"].store}
    if kind == "route":
        idx, w, z = B.smoe_route(ctx, c["top_k"], x=s["x"], w_router=s["w_router"], bias=s["bias"], norm_topk=c["norm_topk"],
                                 want_logits=True)
        return {"idx": idx, "w": w, "logits": z}
    if kind == "prefill":
        y, idx, w, hist = B.smoe_prefill_histogram(ctx, s["routed"], s["shared"], s["x"], c["top_k"], logits=s["logits"],
                                                   w_router=s["w_router"], norm_topk=c["norm_topk"], shared_gate_w=s["gate"],
                                                   add_residual=c["residual"], scratch=s["scratch"])
        return {"y": y, "idx": idx, "w": w, "hist": hist}
    if kind == "ffn":
        B.smoe_expert_ffn(ctx, s["routed"], s["shared"], s["x"], s.get("idx"), s.get("w"), s.get("mask"), add_residual=c["residual"],
                          y=s["y"], prec_out=s["prec"])
        return {"y": s["y"]}
    kw = dict(bias=s["bias"], norm_topk=c["norm_topk"], slice_mask=s["mask"], shared_gate_w=s["gate"], add_residual=c["residual"],
              y=s["y"], idx_out=s["idx"], w_out=s["w"], prec_out=s["prec"])
    if c["tokens"] > 1:
        B.smoe_decode_layer_multi(ctx, s["routed"], s["shared"], s["x"], c["top_k"], s["logits"], **kw)
    else:
        B.smoe_decode_layer(ctx, s["routed"], s["shared"], s["x"], c["top_k"], logits=s["logits"], w_router=s["w_router"], **kw)
    return {"y": s["y"], "idx": s["idx"], "w": s["w"], "prec": s["prec"]}


# ------------------------------------------------------------------------------ unavoidable work
def work(c):
    T, d, E, k, f = c["tokens"], c["d_model"], c["n_experts"], c["top_k"], c["d_ff"]
    ns, fs, G = c["n_shared"], c["shared_d_ff"], c["group"]
    low_bits, esz = NESTS[c["nest"]][1], 4 if c["act"] == "f32" else 2

    def store(ff, planes):                                  # bytes of one expert at so many planes
        meta = 2 * ff * math.ceil(d / G) + d * math.ceil(ff / G)
        return 3 * d * ff * planes * low_bits / 8 + meta * (esz + 1)

    kind = c["kind"]
    if kind == "quantize":
        return {"bytes": E * (3 * d * f * esz + store(f, 2)), "flops": E * 3 * d * f * 4}
    route_b = T * E * 4 * (0 if c["matvec"] else 1) + (E * d * 4 if c["matvec"] else 0) + T * k * 8
    route_f = 2 * T * E * d if c["matvec"] else T * E
    if kind == "route":
        return {"bytes": T * d * esz + route_b + T * E * 4, "flops": route_f}
    act_b = 2 * T * d * esz
    ffn_f = 6 * T * d * (k * f + ns * fs)
    distinct = E * (1.0 - (1.0 - k / E) ** T) if E else 0.0
    if kind == "prefill":
        return {"bytes": act_b + route_b + distinct * store(f, 2) + ns * store(fs, 2), "flops": ffn_f + route_f}
    # decode: about 0.43 of the picks are at both slices under the resident half's bias (1/4 without it)
    p_high = 0.25 if kind == "ffn" else 0.43
    return {"bytes": act_b + (route_b if E else 0) + distinct * store(f, 1 + p_high) + ns * store(fs, 2), "flops": ffn_f + route_f}


def tolerance(c):
    kind = c["kind"]
    if kind == "quantize":
        return "exact"
    if kind == "route":      # fp32 sums of a few thousand terms; near-ties of two scores may swap
        return {"rel": 1e-5, "max": 1e-4, "differ": 1e-3}
    if kind == "prefill":    # bf16 h and y
        return {"rel": 1.5e-2, "max": 0.2, "differ": 1e-3}
    if c["act"] == "f32":
        return {"rel": 1e-5, "max": 1e-4, "differ": 1e-3}
    return {"rel": 8e-3, "max": 5e-2, "differ": 1e-3}      # bf16 y, block-integer activations


# ------------------------------------------------------------------------------ 64-bit reference
def _codes(w, c):
    """Codes [N, K], zero-points and scales [N, groups] of w[N, K] by the fp32 definition of the format."""
    N, K = w.shape
    G, qmax = c["group"], (1 << NESTS[c["nest"]][0]) - 1
    w = w.float()
    ng = -(-K // G)
    wp = torch.zeros((N, ng * G), device=w.device)
    wp[:, :K] = w                                           # (a range always contains 0)
    wg = wp.view(N, ng, G)
    lo, hi = wg.amin(2).clamp(max=0.0), wg.amax(2).clamp(min=0.0)
    half = (qmax + 1) // 2
    # (divisors as tensors: a true division, not a product with the reciprocal)
    s = torch.maximum(hi, -lo) / torch.full_like(hi, half - 1) if c["symmetric"] else (hi - lo) / torch.full_like(hi, qmax)
    if c["act"] == "bf16":
        s = s.bfloat16().float()
    s = torch.where(s > 0, s, torch.ones_like(s))
    zp = torch.full_like(s, half) if c["symmetric"] else torch.round(-lo / s).clamp(0, qmax)
    q = (torch.round(wg / s[:, :, None]) + zp[:, :, None]).clamp(0, qmax)
    return q.reshape(N, ng * G)[:, :K].to(torch.int32), zp.to(torch.int32), s


def _dequant(w, c, high):
    q, zp, s = _codes(w, c)
    K, G, sh = q.shape[1], c["group"], NESTS[c["nest"]][1]
    s, zp = s.double().repeat_interleave(G, 1)[:, :K], zp.repeat_interleave(G, 1)[:, :K]
    return s * (q - zp).double() if high else s * (1 << sh) * ((q >> sh) - (zp >> sh)).double()


def _ffn(x, ws, c, high):
    wg, wu, wd = (_dequant(w, c, high) for w in ws)
    return (torch.nn.functional.silu(x @ wg.T) * (x @ wu.T)) @ wd.T


def _pack_plane(v, bits):
    """One plane (values of `bits` bits, [N, K]) in the store's byte order."""
    N, K = v.shape
    if bits == 4:
        v = v ^ 8
        return (v[:, 0::2] | (v[:, 1::2] << 4)).to(torch.uint8)
    if bits == 2:
        return (v[:, 0::4] | (v[:, 1::4] << 2) | (v[:, 2::4] << 4) | (v[:, 3::4] << 6)).to(torch.uint8)
    v = v.view(N, K // 32, 4, 8).to(torch.int64)            # 6/3: 32 values in three words
    j = torch.arange(8, device=v.device)
    words = torch.zeros((N, K // 32, 3), dtype=torch.int64, device=v.device)
    for t in range(4):
        words[:, :, t >> 1] += ((v[:, :, t] & 3) << (4 * j + 2 * (t & 1))).sum(2)
        words[:, :, 2] += ((v[:, :, t] >> 2) << (4 * j + t)).sum(2)
    return torch.stack([(words >> (8 * b)) & 255 for b in range(4)], 3).reshape(N, K // 32 * 12).to(torch.uint8)


def _exact_store(c, seed):
    E, bits = c["n_experts"], NESTS[c["nest"]][1]
    up = lambda n, m: -(-n // m) * m
    parts = {}                                              # (section, family) -> bytes of all experts
    for e in range(E):
        wg, wu, wd = _dense(c, seed, e)
        for fam, w in (("gu", torch.stack([wg, wu], 1).reshape(2 * c["d_ff"], c["d_model"])), ("dn", wd)):
            q, zp, s = _codes(w, c)
            s = torch.nn.functional.pad(s, (0, s.shape[1] & 1)).to(DT[c["act"]])      # an even number of scales per row
            for sec, t in (("m", _pack_plane(q >> bits, bits)), ("l", _pack_plane(q & ((1 << bits) - 1), bits)),
                           ("z", zp.to(torch.uint8)), ("s", s.contiguous().view(torch.uint8))):
                t = t.reshape(-1)
                if sec in "zs":
                    t = torch.nn.functional.pad(t, (0, up(t.numel(), 16) - t.numel()))
                parts.setdefault((sec, fam), []).append(t)
    out = []
    for sec in "mzsl":
        for fam in ("gu", "dn"):
            t = torch.cat(parts[(sec, fam)])
            out.append(torch.nn.functional.pad(t, (0, up(t.numel(), 256) - t.numel())))
    return {"store": torch.nn.functional.pad(torch.cat(out), (0, 256))}


def exact(c, seed):
    if c["kind"] == "quantize":
        return _exact_store(c, seed)
    s = _inputs(c, seed)
    T, E, k = c["tokens"], c["n_experts"], c["top_k"]
    x = s["x"].double()
    out = {}
    idx = w = prec = None
    if E:
        if c["kind"] == "ffn":
            idx, w = s["idx"].long()[None], s["w"].double()[None]
        else:
            z = s["logits"].double() if s["logits"] is not None else x @ s["w_router"].double().T
            score = z.float() + (0.0 if c["kind"] == "prefill" else s["bias"])
            idx = torch.sort(score, dim=1, descending=True, stable=True)[1][:, :k]
            w = torch.softmax(z, 1).gather(1, idx)
            if c["norm_topk"]:
                w = w / w.sum(1, keepdim=True)
            out = {"idx": idx.to(torch.int32), "w": w}
        if c["kind"] == "route":
            return {**out, "logits": z}
        prec = s["mask"][idx] == 3
        if c["kind"] == "prefill":
            prec = torch.ones_like(prec)
    y = x.clone() if c["residual"] else torch.zeros_like(x)
    if E:
        for e in torch.unique(idx).tolist():
            ws = _dense(c, seed, e)
            t, j = torch.nonzero(idx == e, as_tuple=True)
            for high in (True, False):
                m = prec[t, j] == high
                if bool(m.any()):
                    y.index_add_(0, t[m], w[t[m], j[m]][:, None] * _ffn(x[t[m]], ws, c, high))
    gamma = torch.sigmoid(x @ s["gate"].double())[:, None] if s["gate"] is not None else 1.0
    for e in range(c["n_shared"]):
        y += gamma * _ffn(x, _dense(c, seed, e, shared=True), c, True)
    if c["kind"] == "ffn":
        return {"y": y}
    if c["kind"] == "prefill":
        return {"y": y, **out, "hist": torch.bincount(idx.reshape(-1), minlength=E).to(torch.int32)}
    return {"y": y, **out, "prec": prec.to(torch.uint8)}
