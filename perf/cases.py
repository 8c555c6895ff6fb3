"""The work a program has libkvd do, as timed cases.

Each case is one attention layer's work (the decode step of the 34-layer model
is the one whole call) through the public binding paper_2603_19664_amd.kvd, at
the shapes of this repository's three model configurations:

  op "step"       a KV-Direct decode step: the current token's q, K, V
                  (kvd_project_qkv), then attention over T recomputed context
                  tokens and the current one (kvd_fused_recompute_attn);
                  `layers` layers one after the other, each with its own
                  weights and checkpoints.
  op "window"     the same for a sliding-window layer (kvd_fused_window_attn).
  op "hybrid"     Algorithm 1 with a cache budget: T evicted tokens recomputed,
                  `tail` cached tokens and the current one read from the ring.
  op "cached"     decode attention over stored K/V (kvd_cached_attn, or
                  kvd_decode_attn for the fp32 configuration).
  op "recompute"  RECOMPUTE_KV / prefill: the K/V of T tokens written out.
  op "block"      the block forward of the single-checkpoint scheme.

layout: the weights' memory layout, "row" (row-major), "packed"
(kvd_pack_weights) or "gamma" (kvd_pack_weights_gamma); frozen weights are
packed once, which is part of what a program has in hand.
"""
import math

import torch

from paper_2603_19664_amd import configs, kvd

MODELS = {"smollm": configs.SMOLLM_FP32, "gemma": configs.GEMMA3_4B, "qwen": configs.QWEN_1_5B}
BLOCK_D_FF = 10240  # MLP width of the measured block forward
WINDOW = 1024


def _case(name, op, model, B, T, layout="packed", layers=1, tail=0):
    return {"name": name, "op": op, "model": model, "B": B, "T": T, "layout": layout, "layers": layers, "tail": tail}


def listed():
    return [
        # one decode step of the small fp32 model's layer at its configured context: the smallest call
        _case("smollm_step_fp32", "step", "smollm", 1, 256, "row"),
        # prefill of a ragged prompt in fp32
        _case("smollm_prefill_fp32", "recompute", "smollm", 1, 1000, "row"),
        # one token of the 34-layer model at 4096 tokens of context: the headline decode step
        _case("gemma_step_34_layers", "step", "gemma", 1, 4096, "packed", layers=34),
        # a layer of the batched multi-turn conversation, half way through
        _case("gemma_step_b16", "step", "gemma", 16, 2560),
        # a layer of the long-context batched model
        _case("qwen_step_b8_16k", "step", "qwen", 8, 16384),
        # a sliding-window layer at batch 1: the latency-bound fused call
        _case("gemma_window_b1", "window", "gemma", 1, 4096),
        # a bounded cache of 1024 tokens over 3072 evicted ones
        _case("gemma_hybrid_b8", "hybrid", "gemma", 8, 3072, "gamma", tail=1024),
        # the standard KV-cache decode read at batch 1 and at a batch that fills the memory system
        _case("gemma_cached_b1", "cached", "gemma", 1, 4097),
        _case("gemma_cached_b64", "cached", "gemma", 64, 2049),
        # K/V of a few hundred evicted tokens brought back
        _case("gemma_evicted_256", "recompute", "gemma", 1, 256),
        # prefill of two ragged prompts with weights as a checkpoint stores them
        _case("gemma_prefill_ragged", "recompute", "gemma", 2, 3001, "row"),
        # one block of the single-checkpoint recompute
        _case("gemma_block_4096", "block", "gemma", 1, 4096),
    ]


def draw(rng):
    """One more call from the same ranges: the same operations and models, sizes spread over their logarithm."""
    def logint(lo, hi):
        return max(lo, min(hi, round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))))

    op = rng.choice(["step", "step", "window", "hybrid", "cached", "recompute", "recompute", "block"])
    model = rng.choice({"step": ["smollm", "gemma", "gemma", "qwen", "qwen"], "window": ["gemma", "qwen"],
                        "hybrid": ["gemma", "qwen"], "cached": ["smollm", "gemma", "qwen"],
                        "recompute": ["smollm", "gemma", "qwen"], "block": ["gemma", "qwen"]}[op])
    tail, layout = 0, rng.choice(["row", "packed", "packed", "gamma"])
    if op == "block":
        B = rng.choice([1, 1, 2])
        T = logint(64, 4096 // B)
        layout = rng.choice(["row", "packed"])
    elif model == "smollm":
        B, layout = logint(1, 4), "row"
        T = logint(1, 1024)
    elif op == "cached":
        B = logint(1, 64)
        T = logint(64, 131072 // B)
    elif op == "recompute":
        B = logint(1, 8)
        T = logint(1, 16384 // B)
    else:  # attention over recomputed context
        B = logint(1, 16)
        T = logint(64, (40960 if model == "gemma" else 131072) // B)
        if op == "hybrid":
            tail = logint(4, 2048)
    return {"op": op, "model": model, "B": B, "T": T, "layout": layout, "layers": 1, "tail": tail}


# ---------------------------------------------------------------- inputs

def _inputs(case, seed):
    """The call's tensors as plain torch makes them from the seed: residuals N(0, 1) times the layer's scale,
    weights N(0, 0.02), gamma 1 + N(0, 0.1), in the model's dtype."""
    m = MODELS[case["model"]]
    B, T, L = case["B"], case["T"], case["layers"]
    d, hd, qd, kd = m.d_model, m.head_dim, m.n_q * m.head_dim, m.n_kv * m.head_dim
    dt = torch.bfloat16 if m.dtype == "bf16" else torch.float32
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)

    def normal(shape, std=1.0, mean=0.0):
        return torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32).mul_(std).add_(mean).to(dt)

    lo, hi = m.layer_scale
    x = {"m": m}
    if case["op"] == "cached":
        x["q"] = normal((B, m.n_q, hd))
        x["k"] = normal((B, m.n_kv, T, hd))
        x["v"] = normal((B, m.n_kv, T, hd))
        return x
    x["layers"] = []
    for _ in range(L):
        s = float(torch.rand((), generator=gen, device="cuda")) * (hi - lo) + lo
        w = {"h": normal((B, T, d), s), "h_new": normal((B, d), s), "gamma": normal((d,), m.gamma_std, 1.0),
             "w_q": normal((qd, d), m.w_std), "w_k": normal((kd, d), m.w_std), "w_v": normal((kd, d), m.w_std)}
        if case["op"] == "block":
            f = BLOCK_D_FF
            w.update(w_o=normal((d, qd), m.w_std), gamma_mlp=normal((d,), m.gamma_std, 1.0),
                     w_gate=normal((f, d), m.w_std), w_up=normal((f, d), m.w_std), w_down=normal((d, f), m.w_std))
        x["layers"].append(w)
    if m.pos_offset_max and case["op"] != "window":
        x["pos0"] = torch.randint(0, m.pos_offset_max, (B,), generator=gen, device="cuda", dtype=torch.int32)
    else:
        x["pos0"] = torch.zeros((B,), device="cuda", dtype=torch.int32)
    if case["op"] == "hybrid":  # the cached tokens' K/V, oldest first
        x["tail_k"] = normal((B, m.n_kv, case["tail"], hd))
        x["tail_v"] = normal((B, m.n_kv, case["tail"], hd))
    return x


def _shape(case):
    s = kvd.shape_of(MODELS[case["model"]])
    return {"row": s, "packed": s.packed(), "gamma": s.packed_gamma()}[case["layout"]]


def prepare(case, seed):
    x = _inputs(case, seed)
    m, op, B, T = x["m"], case["op"], case["B"], case["T"]
    s = _shape(case)
    dt, dev = s.torch_dtype, "cuda"
    st = {"op": op, "s": s, "B": B, "T": T, "tail": case["tail"]}
    if op == "cached":
        st.update(q=x["q"], k=x["k"], v=x["v"], out=torch.empty_like(x["q"]),
                  attn=kvd.kvd_cached_attn if m.dtype == "bf16" else kvd.kvd_decode_attn,
                  ws=kvd.workspace(s, kvd.KVD_OP_CACHED_ATTN, B, T))
        return st

    def lay(w, gamma):
        if case["layout"] == "row":
            return w
        return kvd.kvd_pack_weights(s, w) if case["layout"] == "packed" else kvd.kvd_pack_weights_gamma(s, w, gamma)

    layers = []
    for w in x["layers"]:
        y = dict(w)
        for n in ("w_q", "w_k", "w_v"):
            y[n] = lay(w[n], w["gamma"])
        layers.append(y)
    st["layers"], st["pos0"] = layers, x["pos0"]
    if op == "recompute":
        st["k"] = torch.empty((B, m.n_kv, T, m.head_dim), dtype=dt, device=dev)
        st["v"] = torch.empty_like(st["k"])
        return st
    if op == "block":
        w = layers[0]
        if case["layout"] == "packed":
            for n in ("w_o", "w_gate", "w_up", "w_down"):
                w[n] = kvd.kvd_pack_matrix(w[n])
        st["weights"] = kvd.block_weights(w["gamma"], w["w_q"], w["w_k"], w["w_v"], w["w_o"], w["gamma_mlp"],
                                          w["w_gate"], w["w_up"], w["w_down"], s)
        st["out"] = torch.empty((B, T, m.d_model), dtype=dt, device=dev)
        st["ws"] = torch.empty(kvd.kvd_block_workspace_bytes(s, BLOCK_D_FF, B, T), dtype=torch.uint8, device=dev)
        return st
    # decode steps: stacked outputs, one slice a layer; the current token's K/V go into their cache slot
    L, tail = len(layers), case["tail"]
    st["q"] = torch.empty((L, B, m.n_q, m.head_dim), dtype=dt, device=dev)
    st["out"] = torch.empty_like(st["q"])
    st["tk"] = torch.empty((L, B, m.n_kv, tail + 1, m.head_dim), dtype=dt, device=dev)
    st["tv"] = torch.empty_like(st["tk"])
    st["head"] = 0
    if op == "hybrid":  # a ring of tail + 1 slots that has already wrapped: oldest slot `head`, current token before it
        st["head"] = (tail + 1) // 3
        for ring, src in ((st["tk"][0], x["tail_k"]), (st["tv"][0], x["tail_v"])):
            ring[:, :, [(st["head"] + i) % (tail + 1) for i in range(tail)]] = src
    st["slot"] = (st["head"] + tail) % (tail + 1)
    new = min(T + 1, WINDOW) - 1 if op == "window" else T + tail
    st["pos_new"] = st["pos0"] + new
    st["ws"] = kvd.workspace(s, kvd.KVD_OP_FUSED, B, T, tail + 1)
    return st


# ---------------------------------------------------------------- one pass

def run(st):
    op, s, T = st["op"], st["s"], st["T"]
    if op == "cached":
        st["attn"](s, st["q"], st["k"], st["v"], T, st["out"], st["ws"])
        return st["out"]
    if op == "recompute":
        w = st["layers"][0]
        kvd.kvd_recompute_kv(s, w["h"], w["gamma"], w["w_k"], w["w_v"], st["pos0"], T, st["k"], st["v"])
        return st["k"], st["v"]
    if op == "block":
        kvd.kvd_block_forward(s, st["weights"], st["layers"][0]["h"], st["out"], st["pos0"], st["ws"])
        return st["out"]
    for i, w in enumerate(st["layers"]):
        q, out, tk, tv = st["q"][i], st["out"][i], st["tk"][i], st["tv"][i]
        kvd.kvd_project_qkv(s, w["h_new"], w["gamma"], w["w_q"], w["w_k"], w["w_v"], st["pos_new"], q, tk, tv,
                            st["slot"])
        if op == "window":
            kvd.kvd_fused_window_attn(s, q, w["h"], T, w["gamma"], w["w_k"], w["w_v"], WINDOW, out, st["ws"], tk, tv,
                                      1)
        else:
            kvd.kvd_fused_recompute_attn(s, q, w["h"], T, w["gamma"], w["w_k"], w["w_v"], st["pos0"], out, st["ws"],
                                         tk, tv, st["tail"] + 1, st["head"])
    return st["q"], st["tk"], st["tv"], st["out"]


# ---------------------------------------------------------------- cost and accuracy

def work(case):
    """Bytes: every input read once, every output written once.  Flops of attention over recomputed context: the keys'
    projections, the scores, and the values' side as the probability-weighted sum of the residuals followed by one
    projection of it per query head (V is linear in the residual, so no single token's V is needed)."""
    m, op, B, T, L = MODELS[case["model"]], case["op"], case["B"], case["T"], case["layers"]
    e = 2 if m.dtype == "bf16" else 4
    d, hd, qd, kd = m.d_model, m.head_dim, m.n_q * m.head_dim, m.n_kv * m.head_dim
    if op == "cached":
        return {"bytes": e * B * (2 * T * kd + 2 * qd), "flops": 4 * B * T * qd}
    if op == "recompute":
        return {"bytes": e * (B * T * d + 2 * kd * d + d + 2 * B * T * kd), "flops": 4 * B * T * kd * d}
    if op == "block":
        f = BLOCK_D_FF
        mats = d * (qd + 2 * kd) + qd * d + 3 * d * f
        return {"bytes": e * (2 * B * T * d + mats + 2 * d),
                "flops": 2 * B * T * mats + 4 * B * qd * (T * (T + 1) // 2)}
    rec = min(T, WINDOW - 1) if op == "window" else T
    keys = rec + case["tail"] + 1
    flops = 2 * B * d * (qd + 2 * kd) + 2 * B * rec * kd * d + 2 * B * keys * qd + min(
        2 * B * rec * kd * d + 2 * B * keys * qd, 2 * B * rec * m.n_q * d + 2 * B * qd * d + 2 * B * (keys - rec) * qd)
    byts = e * (B * (rec + 1) * d + (qd + 2 * kd) * d + d + 2 * B * kd * (case["tail"] + 1) + 2 * B * qd)
    return {"bytes": L * byts, "flops": L * flops}


def tolerance(case):
    """About four times what the path is off the 64-bit result: fp32 4.4e-7 (the order of the sums); bf16 2.3e-3 to
    2.7e-3 where one rounding of the operands and of the result is all there is (K, V, the block), 4.6e-3 for
    attention over recomputed context (K / V and the probabilities are rounded as well)."""
    if MODELS[case["model"]].dtype == "f32":
        return {"rel": 2e-6}
    return {"rel": 1e-2 if case["op"] in ("recompute", "cached", "block") else 1.8e-2}


def _norm(h, gamma, eps):
    return h * torch.rsqrt(h.square().mean(-1, keepdim=True) + eps) * gamma


def _rope(x, pos, theta):
    """x [..., T, hd], pos [..., T]: consecutive pairs rotated by +pos theta^(-2i / hd)."""
    hd = x.shape[-1]
    f = theta ** (-torch.arange(0, hd, 2, device=x.device, dtype=torch.float64) / hd)
    a = pos.to(torch.float64)[..., None] * f
    c, s = a.cos(), a.sin()
    x0, x1 = x[..., 0::2], x[..., 1::2]
    return torch.stack((x0 * c - x1 * s, x0 * s + x1 * c), -1).flatten(-2)


def _heads(x, w, hd):
    """x [T, d], w [n hd, d] -> [n, T, hd]."""
    return (x @ w.t()).view(x.shape[0], -1, hd).transpose(0, 1)


def _attend(q, k, v):
    """q [n_q, hd], k, v [n_kv, T, hd] -> [n_q, hd]."""
    n_q, hd = q.shape
    g = n_q // k.shape[0]
    q = q.view(k.shape[0], g, hd)
    p = torch.softmax(torch.matmul(q, k.transpose(1, 2).contiguous()) / math.sqrt(hd), -1)
    return torch.matmul(p, v).reshape(n_q, hd)


def _exact_block(x, m, B, T):
    w = {n: t.double() for n, t in x["layers"][0].items()}
    out = torch.empty((B, T, m.d_model), dtype=torch.float64, device="cuda")
    g = m.n_q // m.n_kv
    for b in range(B):
        h = w["h"][b]
        pos = x["pos0"][b] + torch.arange(T, device="cuda")
        hb = _norm(h, w["gamma"], m.rms_eps)
        q = _rope(_heads(hb, w["w_q"], m.head_dim), pos, m.rope_theta)
        k = _rope(_heads(hb, w["w_k"], m.head_dim), pos, m.rope_theta)
        v = _heads(hb, w["w_v"], m.head_dim)
        mask = torch.ones((T, T), dtype=torch.bool, device="cuda").triu(1)
        heads = torch.empty((T, m.n_q, m.head_dim), dtype=torch.float64, device="cuda")
        for i in range(m.n_q):
            s = (q[i] @ k[i // g].t().contiguous() / math.sqrt(m.head_dim)).masked_fill(mask, -math.inf)
            heads[:, i] = torch.softmax(s, -1) @ v[i // g]
        hh = h + heads.reshape(T, -1) @ w["w_o"].t()
        xb = _norm(hh, w["gamma_mlp"], m.rms_eps)
        out[b] = hh + (torch.nn.functional.silu(xb @ w["w_gate"].t()) * (xb @ w["w_up"].t())) @ w["w_down"].t()
    return out


def exact(case, seed):
    x = _inputs(case, seed)
    m, op, B, T, tail = x["m"], case["op"], case["B"], case["T"], case["tail"]
    hd = m.head_dim
    if op == "cached":
        return torch.stack([_attend(x["q"][b].double(), x["k"][b].double(), x["v"][b].double()) for b in range(B)])
    if op == "block":
        return _exact_block(x, m, B, T)
    ks, vs, qs, outs, tks, tvs = [], [], [], [], [], []
    rec0 = T - min(T, WINDOW - 1) if op == "window" else 0
    new = T - rec0 + tail
    for w in x["layers"]:
        gamma, wq, wk, wv = (w[n].double() for n in ("gamma", "w_q", "w_k", "w_v"))
        for b in range(B):
            hb = _norm(w["h"][b, rec0:].double(), gamma, m.rms_eps)
            pos = x["pos0"][b] + torch.arange(T - rec0, device="cuda")
            k = _rope(_heads(hb, wk, hd), pos, m.rope_theta)
            v = _heads(hb, wv, hd)
            if op == "recompute":
                ks.append(k)
                vs.append(v)
                continue
            hn = _norm(w["h_new"][b].double(), gamma, m.rms_eps)[None]
            pn = (x["pos0"][b] + new)[None]
            q = _rope(_heads(hn, wq, hd), pn, m.rope_theta)[:, 0]
            kn = _rope(_heads(hn, wk, hd), pn, m.rope_theta)
            vn = _heads(hn, wv, hd)
            kt, vt = kn, vn
            if op == "hybrid":
                kt = torch.cat((x["tail_k"][b].double(), kn), 1)
                vt = torch.cat((x["tail_v"][b].double(), vn), 1)
            outs.append(_attend(q, torch.cat((k, kt), 1), torch.cat((v, vt), 1)))
            qs.append(q)
            head = (tail + 1) // 3 if op == "hybrid" else 0  # the ring's slots: token i of the tail in slot head + i
            order = [(i - head) % (tail + 1) for i in range(tail + 1)]
            tks.append(kt[:, order])
            tvs.append(vt[:, order])
    if op == "recompute":
        return torch.stack(ks), torch.stack(vs)
    L = len(x["layers"])
    return tuple(torch.stack(t).view(L, B, *t[0].shape) for t in (qs, tks, tvs, outs))
