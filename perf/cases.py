"""The workloads by which the library's speed is followed, through its public
entry points (paper_2608_26574_amd.dard).

Each case is one call as a decoding program makes it: a DARD step of a model
(prefix-cache, full-sequence or shared-prompt form), a prefill or an extend-only
refresh of the prefix cache, the isolated state-masked attention, or the
vocab-wide confidence reduction.  Models have the shapes of synth.py with their
depth cut to a few layers (a layer costs the same whatever its index, and over
a few layers bf16 roundings stay well below the tolerances); weights, prompts
and states are the seeded synthetic ones of synth.py.  exact() evaluates the
same call in float64 with plain torch.
"""
import math

import numpy as np
import torch

from paper_2608_26574_amd import dard, synth

MODELS = {"tiny": synth.TINY, "8b": synth.LLADA8B, "7b": synth.DREAM7B}
TAU_C, TAU_U, LAMBDA, P0 = 0.4, 0.9, 0.5 ** (1 / 8), 0.1
ORDERS = {"confidence": 0, "entropy": dard.F_ORDER_ENTROPY, "left_to_right": dard.F_ORDER_L2R}
M, C, U = 0, 1, 2


# ------------------------------------------------------------------ the cases
def _step(name, model, layers, b, B, P, frac, kv="", mix="logits", order="confidence", Ps=0):
    return {"name": name, "kind": "step", "model": model, "layers": layers, "b": b, "B": B, "P": P, "frac": frac,
            "kv": kv, "mix": mix, "order": order, "Ps": Ps}


def listed():
    return [
        # the smallest whole step: a two-layer fp32 model, one 32-token block
        _step("step_tiny_f32", "tiny", 2, 1, 32, 64, 0.25),
        # latency-bound decoding of one sequence, the middle of a generation (prompt 512, fourth block)
        _step("step_8b_b1", "8b", 3, 1, 32, 608, 0.25),
        # a few sequences served together, prompt of an arbitrary length
        _step("step_8b_b3_ragged", "8b", 3, 3, 32, 535, 0.25),
        # throughput decoding with grouped-query attention, blocks of 64
        _step("step_7b_b8", "7b", 2, 8, 64, 1216, 0.3),
        # many multimodal sequences (576 image + 256 text positions), hidden-state mixing
        _step("step_8b_b32_hidden", "8b", 2, 32, 32, 832, 0.3, mix="hidden"),
        # a step without a prefix cache: 256 prompt + 256 generated positions, the first block of 128
        {"name": "step_full_8b", "kind": "full", "model": "8b", "layers": 2, "b": 1, "B": 128, "N": 512, "blk": 256,
         "frac": 0.25},
        # the exact refresh of the prefix cache at a block boundary, an odd prompt length
        {"name": "prefill_8b_b1", "kind": "prefill", "model": "8b", "layers": 2, "b": 1, "P": 651},
        # the prompts of a batch
        {"name": "prefill_7b_b8", "kind": "prefill", "model": "7b", "layers": 2, "b": 8, "P": 1024},
        # the extend-only refresh: one committed block of each of four sequences
        {"name": "extend_8b_b4", "kind": "extend", "model": "8b", "layers": 2, "b": 4, "P": 576, "Pn": 32},
        # the isolated attention: the grouped-query shape, and the multi-head one with an FP8 KV cache
        {"name": "attention_gqa_b8", "kind": "attention", "Hq": 28, "Hkv": 4, "b": 8, "B": 64, "P": 1472, "frac": 0.3,
         "kv": ""},
        {"name": "attention_mha_b16_fp8", "kind": "attention", "Hq": 32, "Hkv": 32, "b": 16, "B": 32, "P": 512,
         "frac": 0.25, "kv": "fp8"},
        # the confidence reduction over a batch's masked positions, mixed logits
        {"name": "confidence_7b", "kind": "confidence", "rows": 360, "V": 152064, "mix": "logits", "stats": False},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step"] * 5 + ["full", "prefill", "prefill", "extend", "attention", "attention", "confidence"])
    if kind == "attention":
        Hq, Hkv = rng.choice([(32, 32), (28, 4)])
        return {"kind": kind, "Hq": Hq, "Hkv": Hkv, "b": _log(rng, 1, 16), "B": rng.choice([16, 24, 32, 48, 64, 128]),
                "P": _log(rng, 64, 2048), "frac": rng.choice([0.1, 0.25, 0.5]), "kv": rng.choice(["", "", "fp8"])}
    if kind == "confidence":
        return {"kind": kind, "rows": _log(rng, 8, 1024), "V": rng.choice([2048, 126464, 152064]),
                "mix": rng.choice(["", "logits"]), "stats": rng.random() < 0.3}
    if kind == "full":
        B = rng.choice([32, 64, 128, 256])
        N = B * rng.randint(1, 3) + rng.randint(32, 400)
        return {"kind": kind, "model": "8b", "layers": rng.randint(1, 2), "b": rng.randint(1, 2), "B": B, "N": N,
                "blk": rng.randint(0, N - B), "frac": rng.choice([0.1, 0.25, 0.5])}
    model = rng.choice(["tiny", "8b", "8b", "7b"])
    layers = rng.randint(1, 2)
    if kind == "prefill":
        b = _log(rng, 1, 8)
        return {"kind": kind, "model": model, "layers": layers, "b": b,
                "P": _log(rng, 64, 256 if model == "tiny" else min(2048, 8192 // b))}
    if kind == "extend":
        return {"kind": kind, "model": model, "layers": layers, "b": _log(rng, 1, 16), "P": _log(rng, 64, 1024),
                "Pn": rng.choice([16, 32, 48, 64])}
    if model == "tiny":
        return _drawn(rng, "tiny", layers, rng.randint(1, 3), rng.choice([16, 24, 32]), _log(rng, 32, 256), "", 0)
    b, B = _log(rng, 1, 16), rng.choice([16, 24, 32, 37, 64])
    P = _log(rng, 128, 1472)
    # (over more layers the FP8 cache's roundings grow past any useful tolerance)
    kv = rng.choice(["", "", "fp8"]) if layers == 1 else ""
    return _drawn(rng, model, layers, b, B, P, kv, P // 128 * 64 if rng.random() < 0.2 else 0)


def _drawn(rng, model, layers, b, B, P, kv, Ps):
    c = _step("", model, layers, b, B, P, rng.choice([0.1, 0.25, 0.3, 0.5]), kv, rng.choice(["logits", "logits", "hidden"]),
              rng.choice(["confidence", "confidence", "entropy", "left_to_right"]), Ps)
    del c["name"]
    return c


# ------------------------------------------------------------------ what a program has before the call
def _dims(c):
    d = MODELS[c["model"]].as_dict()
    d["n_layers"] = c["layers"]
    d["kv_dtype"] = c.get("kv", "")
    return synth.Dims(**d)


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _ids(c, n, V, seed):
    return _dev(synth.prompt_ids(c["b"], n, V, seed=seed))


def _block(c, V, seed):
    """(tokens, states, confidences) of the current block of every sequence."""
    return tuple(_dev(a) for a in synth.workload_block(c["b"], c["B"], c["frac"], V, seed=seed, tau_c=TAU_C, tau_u=TAU_U))


def _inputs(c, seed):
    """The raw inputs of a case, from its seed alone (shared by prepare and exact)."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    if c["kind"] == "confidence":
        rows, V = c["rows"], c["V"]
        std = 1.3   # of the logits of the random-init heads
        x = {"s": torch.randn(rows, V, generator=g, device="cuda") * std}
        if c["mix"]:
            x["x"] = torch.randn(rows, V, generator=g, device="cuda") * std
            x["w"] = torch.rand(rows, generator=g, device="cuda")
        return x
    if c["kind"] == "attention":
        b, B, P, Hq, Hkv, dh = c["b"], c["B"], c["P"], c["Hq"], c["Hkv"], 128
        cap = P + 2 * B
        q = torch.randn(b, 2 * B, Hq, dh, generator=g, device="cuda").bfloat16()
        k = torch.randn(b, Hkv, cap, dh, generator=g, device="cuda")
        v = torch.randn(b, Hkv, dh, cap, generator=g, device="cuda")
        if c["kv"] == "fp8":
            k, v = (t.to(torch.float8_e4m3fn).view(torch.uint8) for t in (k, v))
        else:
            k, v = k.bfloat16(), v.bfloat16()
        _, state, conf = _block(c, 1 << 15, seed + 1)
        return {"q": q, "k": k, "v": v, "state": state, "conf": conf}
    dims = _dims(c)
    V = dims.vocab
    x = {"dims": dims, "weights": synth.make_weights(dims, seed=seed + 2, device="cuda")}
    if c["kind"] == "prefill":
        x["ids"] = _ids(c, c["P"], V, seed + 3)
        return x
    if c["kind"] == "extend":
        x["ids"] = _ids(c, c["P"], V, seed + 3)
        x["new"] = _ids(c, c["Pn"], V, seed + 4)
        return x
    x["tok"], x["state"], x["conf"] = _block(c, V, seed + 4)
    if c["kind"] == "full":
        seq = _ids(c, c["N"], V, seed + 3)
        seq[:, c["blk"]:c["blk"] + c["B"]] = x["tok"]
        seq[:, c["blk"] + c["B"]:] = dims.mask_id
        x["seq"] = seq
        return x
    if c["Ps"]:
        x["ids"] = _ids({"b": 1}, c["Ps"], V, seed + 3)
        x["own"] = _ids(c, c["P"] - c["Ps"], V, seed + 5)
    else:
        x["ids"] = _ids(c, c["P"], V, seed + 3)
        if c["b"] >= 16 and c["P"] > 576:   # multimodal prompts open with 576 embedding positions
            x["embeds"] = torch.randn(c["b"], c["P"], dims.d_model, generator=g, device="cuda").to(synth.torch_dtype(dims))
            x["ids"][:, :576] = -1
    return x


def _cap(c):
    return {"prefill": c.get("P", 0) + 64, "extend": c.get("P", 0) + c.get("Pn", 0) + 64,
            "full": c.get("N", 0) + c.get("B", 0)}.get(c["kind"], c.get("P", 0) + 2 * c.get("B", 0) + 32)


def prepare(c, seed):
    x = _inputs(c, seed)
    if c["kind"] == "confidence":
        n = c["rows"]
        f = lambda: torch.zeros(n, device="cuda")   # noqa: E731
        x.update(argmax=torch.zeros(n, dtype=torch.int32, device="cuda"), maxprob=f(), entropy=f() if c["stats"] else None,
                 margin=f() if c["stats"] else None,
                 ws=torch.empty(dard.dard_confidence_workspace_bytes(n, c["V"]), dtype=torch.uint8, device="cuda"))
        return {"c": c, **x}
    if c["kind"] == "attention":
        x["out"] = torch.empty_like(x["q"])
        dt = dard.DTYPE_BF16_KV_FP8 if c["kv"] == "fp8" else dard.DTYPE_BF16
        x["ws"] = torch.empty(dard.dard_attention_workspace_bytes(dt, c["b"], c["B"], c["Hq"], 128, c["P"]),
                              dtype=torch.uint8, device="cuda")
        return {"c": c, **x}
    dims, b, B, cap = x["dims"], c["b"], c.get("B", 16), _cap(c)
    eng = dard.Engine(dims, x.pop("weights"), b, B, cap)
    s = {"c": c, "eng": eng, **x}
    if c["kind"] in ("prefill", "extend"):
        if c["kind"] == "extend":
            eng.dard_prefill(s["ids"])
        return s
    flags = (dard.F_HIDDEN_MIX if c.get("mix") == "hidden" else 0) | ORDERS[c.get("order", "confidence")]
    s["params"] = dard.make_params(tau_c=TAU_C, tau_u=TAU_U, lam=LAMBDA, p0=P0, mask_id=dims.mask_id, flags=flags)
    i32 = dict(dtype=torch.int32, device="cuda")
    s["out"] = {"tok": torch.zeros(b, B, **i32), "state": torch.zeros(b, B, dtype=torch.uint8, device="cuda"),
                "conf": torch.zeros(b, B, device="cuda"), "done": torch.zeros(b, **i32),
                # rows that the LM head does not run over stay zero
                "logits": torch.zeros(b, 2 * B, dims.vocab, device="cuda")}
    if c["kind"] == "step":
        if c["Ps"]:
            s["shared"] = dard.Engine(dims, None, 1, B, max(c["Ps"], 2 * B), packed=eng.packed)
            s["shared"].dard_prefill(s["ids"])
            if c["P"] > c["Ps"]:
                eng.dard_prefill_suffix(s["shared"], c["Ps"], s["own"])
        else:
            eng.dard_prefill(s["ids"], embeds=s.get("embeds"))
    return s


# ------------------------------------------------------------------ one pass
def run(s):
    c = s["c"]
    if c["kind"] == "confidence":
        dard.dard_confidence(s["s"], s["argmax"], s["maxprob"], logits_x=s.get("x"), w=s.get("w"), ws=s["ws"],
                             entropy=s["entropy"], margin=s["margin"])
        return {k: s[k] for k in ("argmax", "maxprob", "entropy", "margin")}
    if c["kind"] == "attention":
        dard.dard_masked_attention(s["q"], s["k"], s["v"], c["P"], s["state"], s["conf"], 128 ** -0.5, 0, s["out"],
                                   ws=s["ws"])
        return s["out"]
    eng = s["eng"]
    if c["kind"] in ("prefill", "extend"):
        if c["kind"] == "prefill":
            eng.dard_prefill(s["ids"])
        else:
            eng.dard_prefill_extend(c["P"], s["new"])
        return dict(zip("kv", eng.kv_view(synth.torch_dtype(eng.dims))))
    o = s["out"]
    outs = (o["tok"], o["state"], o["conf"], o["done"])
    if c["kind"] == "full":
        eng.dard_step_full(c["blk"], s["params"], s["seq"], s["state"], s["conf"], *outs, debug={"logits": o["logits"]})
    elif c["Ps"]:
        eng.dard_step_shared(s["shared"], c["Ps"], c["P"], s["params"], s["tok"], s["state"], s["conf"], *outs,
                             debug={"logits": o["logits"]})
    else:
        eng.dard_step(c["P"], s["params"], s["tok"], s["state"], s["conf"], *outs, debug={"logits": o["logits"]})
    return o


# ------------------------------------------------------------------ what a pass cannot do without
def work(c):
    if c["kind"] == "confidence":
        n = c["rows"] * c["V"] * (2 if c["mix"] else 1)
        return {"bytes": 4 * n + 8 * c["rows"], "flops": 4 * n}
    if c["kind"] == "attention":
        b, B, P, Hq, Hkv, dh = c["b"], c["B"], c["P"], c["Hq"], c["Hkv"], 128
        kv = 1 if c["kv"] == "fp8" else 2
        return {"bytes": 2 * b * Hkv * (P + 2 * B) * dh * kv + 2 * b * 2 * B * Hq * dh * 2,
                "flops": 4 * b * 2 * B * Hq * (P + B) * dh}
    d = _dims(c)
    es = 2 if d.dtype == "bf16" else 4
    kves = 1 if d.kv_dtype == "fp8" else es
    kd = d.n_kv_heads * d.head_dim
    per_layer = d.d_model * (2 * d.d_model + 2 * kd) + 3 * d.d_model * d.ffn_dim   # weights
    b, B = c["b"], c.get("B", 0)
    # token rows, keys that each of them attends to, cached keys read
    rows, keys, cached = {"prefill": (b * c.get("P", 0), c.get("P", 0), 0),
                          "extend": (b * c.get("Pn", 0), c.get("P", 0) + c.get("Pn", 0), b * c.get("P", 0)),
                          "full": (b * (c.get("N", 0) + B), c.get("N", 0), 0),
                          "step": (b * 2 * B, c.get("P", 0) + B, b * (c.get("P", 0) - c.get("Ps", 0)) + c.get("Ps", 0)),
                          }[c["kind"]]
    nbytes = d.n_layers * (per_layer * es + 2 * kd * kves * (cached + rows)) + rows * d.d_model * es
    flops = d.n_layers * (2 * rows * per_layer + 4 * rows * keys * d.d_model)
    if c["kind"] in ("step", "full"):
        n_c = int(round(c["frac"] * B))
        head = b * (B + int(math.ceil((B - n_c) / 2)))   # shadow rows, and the x rows of masked positions
        nbytes += d.vocab * d.d_model * es + 4 * head * d.vocab
        flops += 2 * head * d.vocab * d.d_model
    return {"bytes": nbytes, "flops": flops}


def tolerance(c):
    if c["kind"] == "confidence":
        return {"rel": 5e-6}                # fp32 sums over the vocabulary (3e-7 from float64)
    if c["kind"] == "attention":
        return {"rel": 1e-2}                # bf16 probabilities and outputs (2.3e-3 from float64)
    if c["model"] == "tiny":
        return {"rel": 5e-6}                # fp32 throughout (8e-7 from float64)
    if c["kind"] in ("prefill", "extend"):
        return {"rel": 2e-2, "max": 0.5}    # bf16 activations through every layer (6.8e-3 from float64)
    return {"rel": 3e-2, "max": 0.5, "differ": 0.01}   # (7e-3 to 1.5e-2 over two to four layers)


# ------------------------------------------------------------------ the same calls in float64
def _take_x(state, conf, order):
    """[b][2B][B]: does the row (x rows, then shadow rows) read x^j (else s^j)?"""
    b, B = state.shape
    u, cand = (state == U)[:, None, :], (state == C)[:, None, :]
    if order == "left_to_right":
        before = (torch.arange(B, device=state.device)[None, None, :] <= torch.arange(B, device=state.device)[None, :, None])
    else:
        before = conf[:, :, None] <= conf[:, None, :]
    me = torch.eye(B, dtype=torch.bool, device=state.device)[None]
    si = state[:, :, None]
    by_cand = u | (cand & before)
    x = torch.where(si == U, u, torch.where(si == C, by_cand, torch.ones_like(by_cand)))
    s = torch.where(si == C, by_cand, u.expand(b, B, B)) & ~me
    s = torch.where(si == M, u.expand(b, B, B), s)
    return torch.cat([x, s], 1)


def _attend(q, k, v, visible, scale):
    """q [b][R][Hq][dh], k / v [b][K][Hkv][dh], visible [b][R][K] or None (every key)."""
    b, R, Hq, dh = q.shape
    Hkv = k.shape[2]
    out = torch.empty_like(q)
    for i in range(b):
        for h in range(Hkv):
            hs = slice(h * (Hq // Hkv), (h + 1) * (Hq // Hkv))
            qh = q[i, :, hs].reshape(-1, dh)                                    # rows x heads of the group
            sc = qh @ k[i, :, h].T * scale
            if visible is not None:
                sc = sc.masked_fill(~visible[i].repeat_interleave(Hq // Hkv, 0), -math.inf)
            out[i, :, hs] = (torch.softmax(sc, -1) @ v[i, :, h]).reshape(R, -1, dh)
    return out


def _rope(x, pos, theta):
    """Rotate-half; x [b][R][H][dh], pos [R]."""
    half = x.shape[-1] // 2
    ang = pos.double()[:, None] * theta ** (-2.0 * torch.arange(half, device=x.device).double() / x.shape[-1])
    cos, sin = torch.cos(ang)[:, None], torch.sin(ang)[:, None]
    a, z = x[..., :half], x[..., half:]
    return torch.cat([a * cos - z * sin, z * cos + a * sin], -1)


def _stored(x, dims):
    """The cached value of x: the FP8 format is part of the call, other types store x itself."""
    if dims.kv_dtype != "fp8":
        return x
    return x.float().clamp(-448, 448).to(torch.float8_e4m3fn).double()


def _norm(h, gain, eps):
    return h / torch.sqrt((h * h).mean(-1, keepdim=True) + eps) * gain.double()


def _forward(w, dims, h, pos, visible, past):
    """The layers over rows h [b][R][d]; past: per layer (k, v) [b][P][Hkv][dh] in front of the
    rows' own keys, or None.  Returns the final-normalised rows and every layer's own (k, v)."""
    b, R, _ = h.shape
    dh, own = dims.head_dim, []
    for l in range(dims.n_layers):
        p = "layers.%d." % l
        W = lambda name: w[p + name].double()   # noqa: E731
        xn = _norm(h, w[p + "attn_norm"], dims.norm_eps)
        q = _rope((xn @ W("wq").T).view(b, R, -1, dh), pos, dims.rope_theta)
        k = _stored(_rope((xn @ W("wk").T).view(b, R, -1, dh), pos, dims.rope_theta), dims)
        v = _stored((xn @ W("wv").T).view(b, R, -1, dh), dims)
        own.append((k, v))
        if past is not None:
            k, v = (torch.cat([o.expand(b, -1, -1, -1), n], 1) for o, n in zip(past[l], (k, v)))
        h = h + _attend(q, k, v, visible, dh ** -0.5).reshape(b, R, -1) @ W("wo").T
        xn = _norm(h, w[p + "ffn_norm"], dims.norm_eps)
        for at in range(0, R, 512):   # the feed-forward width times all rows need not be held at once
            part = xn[:, at:at + 512]
            h[:, at:at + 512] += (torch.nn.functional.silu(part @ W("w_gate").T) * (part @ W("w_up").T)) @ W("w_down").T
    return _norm(h, w["final_norm"], dims.norm_eps), own


def _embed(w, ids, embeds=None):
    h = w["embed"][ids.clamp(min=0).long()].double()
    return h if embeds is None else torch.where((ids < 0)[..., None], embeds.double(), h)


def _decisions(c, dims, w, xn, state):
    """Logits of the rows that the decisions read (others zero) and the confidences carried on."""
    b, B = state.shape
    V = dims.vocab
    head = w["lm_head"].double()
    x, s = xn[:, :B], xn[:, B:]
    ls = s @ head.T
    all_rows = dims.dtype == "bf16" and b * 2 * B <= 64 and c.get("mix") != "hidden"

    def top(l):
        return 1.0 / torch.exp(l - l.amax(-1, keepdim=True)).sum(-1)

    conf = top(ls)
    up, down = (state == C) & (conf > TAU_U), (state == C) & (conf <= TAU_C)
    i = torch.arange(B, device=state.device)
    kern = LAMBDA ** (i[:, None] - i[None]).abs().double()
    p, d = up.double() @ kern, down.double() @ kern
    wt = ((p + P0) / (p + d + P0))[..., None]
    masked = (state == M)[..., None]
    if c.get("mix") == "hidden":
        s = torch.where(masked, wt * x + (1 - wt) * s, s)
        lm = ls = s @ head.T
        lx = torch.zeros(1, dtype=ls.dtype, device=ls.device).expand_as(ls)
    else:
        lx = x @ head.T
        lm = torch.where(masked, wt * lx + (1 - wt) * ls, ls)
        if not all_rows:
            lx = lx * masked
    conf = top(lm)
    if c.get("order") == "entropy":
        lp = torch.log_softmax(lm, -1)
        conf = (lp.exp() * lp).sum(-1)
    return {"tok": None, "state": None, "conf": conf, "done": None, "logits": torch.cat([lx, ls], 1).view(b, 2 * B, V)}


def exact(c, seed):
    x = _inputs(c, seed)
    if c["kind"] == "confidence":
        l = x["s"].double()
        if c["mix"]:
            w = x["w"].double()[:, None]
            l = w * x["x"].double() + (1 - w) * l
        m2 = l.topk(2, -1).values
        p = torch.exp(l - m2[:, :1])
        s = p.sum(-1)
        lp = l - m2[:, :1] - s.log()[:, None]
        return {"argmax": None, "maxprob": 1 / s, "entropy": -(p / s[:, None] * lp).sum(-1) if c["stats"] else None,
                "margin": (1 - torch.exp(m2[:, 1] - m2[:, 0])) / s if c["stats"] else None}
    if c["kind"] == "attention":
        k, v = x["k"], x["v"]
        if c["kv"] == "fp8":
            k, v = (t.view(torch.float8_e4m3fn) for t in (k, v))
        take = _take_x(x["state"], x["conf"], "confidence")
        seen = torch.cat([torch.ones(*take.shape[:2], c["P"], dtype=torch.bool, device="cuda"), take, ~take], -1)
        return _attend(x["q"].double(), k.double().transpose(1, 2), v.double().permute(0, 3, 1, 2), seen, 128 ** -0.5)
    dims, w, b, B = x["dims"], x["weights"], c["b"], c.get("B", 0)
    at = lambda lo, hi: torch.arange(lo, hi, device="cuda")   # noqa: E731
    if c["kind"] in ("prefill", "extend"):
        _, kv = _forward(w, dims, _embed(w, x["ids"]), at(0, c["P"]), None, None)
        if c["kind"] == "extend":
            _, new = _forward(w, dims, _embed(w, x["new"]), at(c["P"], c["P"] + c["Pn"]), None, kv)
            kv = [tuple(torch.cat(t, 1) for t in zip(o, n)) for o, n in zip(kv, new)]
        # the cache holds each head's K dims in the order 0, dh/2, 1, dh/2 + 1, ..., zeros past the last key
        pairs = torch.arange(dims.head_dim, device="cuda").view(2, -1).T.reshape(-1)
        pad = lambda t: torch.nn.functional.pad(t.transpose(1, 2), (0, 0, 0, _cap(c) - t.shape[1]))   # noqa: E731
        return {"k": torch.stack([pad(k[..., pairs]) for k, _ in kv]), "v": torch.stack([pad(v) for _, v in kv])}
    take = _take_x(x["state"], x["conf"], c.get("order", "confidence"))
    shadow = torch.full((b, B), dims.mask_id, device="cuda")
    if c["kind"] == "full":
        # rows and keys: the sequence, then the shadow block; only the block's rows read by state
        N, blk = c["N"], c["blk"]
        seen = torch.ones(b, N + B, N + B, dtype=torch.bool, device="cuda")
        seen[:, :, N:] = False
        for rows, part in ((slice(blk, blk + B), take[:, :B]), (slice(N, N + B), take[:, B:])):
            seen[:, rows, blk:blk + B] = part
            seen[:, rows, N:] = ~part
        pos = torch.cat([at(0, N), at(blk, blk + B)])
        xn, _ = _forward(w, dims, _embed(w, torch.cat([x["seq"], shadow], 1)), pos, seen, None)
        xn = torch.cat([xn[:, blk:blk + B], xn[:, N:]], 1)
        return _decisions(c, dims, w, xn, x["state"])
    _, past = _forward(w, dims, _embed(w, x["ids"], x.get("embeds")), at(0, x["ids"].shape[1]), None, None)
    if c["Ps"]:
        past = [tuple(t.expand(b, -1, -1, -1) for t in kv) for kv in past]
        if c["P"] > c["Ps"]:
            _, own = _forward(w, dims, _embed(w, x["own"]), at(c["Ps"], c["P"]), None, past)
            past = [tuple(torch.cat(t, 1) for t in zip(o, n)) for o, n in zip(past, own)]
    seen = torch.cat([torch.ones(b, 2 * B, c["P"], dtype=torch.bool, device="cuda"), take, ~take], -1)
    pos = torch.cat([at(c["P"], c["P"] + B)] * 2)
    xn, _ = _forward(w, dims, _embed(w, torch.cat([x["tok"], shadow], 1)), pos, seen, past)
    return _decisions(c, dims, w, xn, x["state"])
