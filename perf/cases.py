"""Performance cases of the packed prefill and the generation that follows it.

Each case is one pass through the library's public entry points, with weights, plan, caches and
workspaces resident as a serving program keeps them:

  prefill      the prompts of a batch to their hidden states, caches and first-token logits
               (pp_prefill, then pp_first_token), bf16 models and the small float32 one
  qkv          attention norm and QKV projection of one layer (pp_rmsnorm, pp_qkv_projection)
  mlp          MLP norm, gate/up and down projections of one layer (pp_rmsnorm, pp_gemm twice)
  attention    attention of one layer over a packed batch (pp_attention)
  decode       one generated token of every prompt (pp_decode_step)
  first_token  LM head and greedy choice on every prompt's last hidden row (pp_first_token)

A case is described by its model shape, its prompt count and the length mix of its prompts (a
workload id of ``workloads.py``, or 0 for nine one-token prompts to every one of a thousand);
the lengths follow from the case alone, so its work is known without drawing the inputs.
"""
import math
import types

import numpy as np
import torch

from paper_2404_09529_amd import prepack as pp
from paper_2404_09529_amd import workloads as W

DEV = "cuda"
SHAPES = {
    "tiny-f32": W.WORKLOADS[1].shape,                     # d 256, 4 heads of 64, F 688, float32
    "tiny-f32-gqa": W.WORKLOADS[1].shape.replace(n_kv_heads=2),
    "1.3b": W.MODELS["llama-1.3b"],                       # d 2048, 16 heads, F 5504
    "7b": W.MODELS["llama2-7b"],                          # d 4096, 32 heads, F 11008
    "7b-gqa": W.MODELS["mistral-7b"],                     # d 4096, 32/8 heads, F 14336
    "8b-gqa": W.WORKLOADS[4].shape,                       # the same with vocabulary 128256, theta 5e5
    "13b": W.MODELS["llama2-7b"].replace(d_model=5120, n_heads=40, n_kv_heads=40, ffn_dim=13824),
}
N_NEW, STEP = 24, 17   # decode: room for 24 generated tokens per prompt, the 18th being generated


def listed():
    return [
        # the smallest call: a toy float32 model, 8 prompts of 4-64 tokens; launches and latency
        dict(name="prefill-tiny-f32", path="prefill", shape="tiny-f32", layers=1, k=8, lengths=1, seed=0, row=128),
        # an interactive request or two at a small model: a few hundred tokens, weights dominate
        dict(name="prefill-1.3b-2-prompts", path="prefill", shape="1.3b", layers=2, k=2, lengths=12, seed=1, row=0),
        # the evaluation batch of 16 dataset prompts (mean 169 tokens), grouped-query 7B layer
        dict(name="prefill-7b-gqa-16-prompts", path="prefill", shape="7b-gqa", layers=1, k=16, lengths=12, seed=0, row=0),
        # the throughput batch: 64 prompts, 27.7k tokens in rows of 4096
        dict(name="prefill-7b-64-prompts", path="prefill", shape="7b", layers=1, k=64, lengths=2, seed=0, row=4096),
        # one layer's MLP for 16 short prompts (mean 73 tokens) of a small model
        dict(name="mlp-1.3b-16-prompts", path="mlp", shape="1.3b", k=16, lengths=7, seed=0, row=0),
        # one layer's norm and QKV projection for 16 chat prompts (mean 247 tokens), 13B width
        dict(name="qkv-13b-16-prompts", path="qkv", shape="13b", k=16, lengths=10, seed=0, row=0),
        # attention over 64 mostly short prompts
        dict(name="attention-7b-64-prompts", path="attention", shape="7b", k=64, lengths=2, seed=0, row=4096),
        # attention with grouped heads over longer prompts (up to 8192 tokens)
        dict(name="attention-8b-gqa-long", path="attention", shape="8b-gqa", k=48, lengths=4, seed=0, row=8192),
        # generation for the paper's toy batch: nine 1-token prompts and one of 1000
        dict(name="decode-7b-10-prompts", path="decode", shape="7b", layers=2, k=10, lengths=0, seed=0),
        # serving a grouped-query model: 48 chats in flight
        dict(name="decode-7b-gqa-48-prompts", path="decode", shape="7b-gqa", layers=2, k=48, lengths=10, seed=0),
        # serving a small model at high concurrency: 150 prompts of up to 512 tokens
        dict(name="decode-1.3b-150-prompts", path="decode", shape="1.3b", layers=2, k=150, lengths=6, seed=0),
        # first token of 64 prompts over a large vocabulary
        dict(name="first-token-8b-64-prompts", path="first_token", shape="8b-gqa", k=64, lengths=8, seed=0, row=0),
    ]


def _cost(case):
    w = work(case)
    return max(w["bytes"] / 4e12, w["flops"] / 1e15)


def draw(rng):
    """One more case of the same ranges: any path, shape, length mix and prompt count whose work
    is at most the largest listed case's."""
    most = max(_cost(c) for c in listed())
    while True:
        path = rng.choice(["prefill", "prefill", "qkv", "mlp", "attention", "decode", "decode", "first_token"])
        shape = rng.choice(["1.3b", "7b", "7b-gqa", "8b-gqa", "13b"])
        if path == "prefill" and rng.random() < 0.25:
            shape = rng.choice(["tiny-f32", "tiny-f32-gqa"])
        f32 = shape.startswith("tiny")
        case = dict(path=path, shape=shape, seed=rng.randrange(1000))
        top = 48 if f32 else {"decode": 256, "first_token": 200, "attention": 96}.get(path, 64)
        case["k"] = int(round(math.exp(rng.uniform(0.0, math.log(top)))))
        case["lengths"] = 1 if f32 else rng.choice([0, 2, 4, 6, 7, 8, 9, 10, 11, 12] + ([5] if path == "attention" else []))
        if path in ("prefill", "decode"):
            case["layers"] = rng.choice([1, 2])
        if path != "decode":
            m = int(lengths_of(case).max())
            case["row"] = rng.choice([0, m + rng.randrange(1, 400), 2 * m + 1])
        if _cost(case) <= most:
            return case


# ----------------------------------------------------------------------------- sizes
def lengths_of(case):
    k = case["k"]
    if case["lengths"] == 0:
        out = np.ones(k, dtype=np.int32)
        out[k // 2::10] = 1000
        return out
    return W.draw_lengths(W.workload(case["lengths"]), case["seed"], k)


def _shape(case):
    return SHAPES[case["shape"]].replace(n_layers=case.get("layers", 1))


def work(case):
    s, n = _shape(case), lengths_of(case).astype(np.int64)
    L, k, e = int(n.sum()), int(n.size), 2 if s.dtype == "bf16" else 4
    d, F, V = s.d_model, s.ffn_dim, s.vocab
    hd, kvw = s.n_heads * s.head_dim, s.n_kv_heads * s.head_dim
    per_layer = d * (hd + 2 * kvw) + hd * d + 3 * d * F       # weights
    pairs = int((n * (n + 1) // 2).sum())
    path = case["path"]
    if path == "prefill":
        by = s.n_layers * (per_layer * e + 2 * L * kvw * e) + L * d * (e + 4) + V * d * e + k * V * 4
        fl = s.n_layers * (2 * L * per_layer + 4 * pairs * hd) + 2 * k * V * d
    elif path == "qkv":
        by, fl = d * (hd + 2 * kvw) * e + L * d * 4 + L * (hd + 2 * kvw) * e, 2 * L * d * (hd + 2 * kvw)
    elif path == "mlp":
        by, fl = 3 * d * F * e + L * d * 8 + L * F * e, 6 * L * d * F
    elif path == "attention":
        by, fl = 2 * L * (hd + kvw) * e, 4 * pairs * hd
    elif path == "decode":
        keys = L + k * (STEP + 1)
        by = s.n_layers * (per_layer * e + 2 * keys * kvw * e) + V * d * e + k * d * e + k * V * 4
        fl = s.n_layers * (2 * k * per_layer + 4 * keys * hd) + 2 * k * V * d
    else:
        by, fl = V * d * e + k * d * 4 + k * V * 4, 2 * k * V * d
    return {"bytes": by, "flops": fl}


def tolerance(case):
    # float32 sums in another order differ by about 5e-7.  bf16 results are off their 64-bit values
    # by the storage's rounding: 2.3e-3 measured for qkv, 2.9e-3 for mlp, 2.0e-3 for attention
    # (whose probabilities may be scaled differently before they are rounded), 9e-3 through a
    # whole call; two correct implementations by up to sqrt(2) of that
    if _shape(case).dtype == "f32" or case["path"] == "first_token":
        return {"rel": 1e-5, "max": 1e-3}
    return {"rel": {"qkv": 4e-3, "mlp": 6e-3, "attention": 8e-3}.get(case["path"], 2e-2)}


# ----------------------------------------------------------------------------- inputs
def _generator(seed):
    return torch.Generator(device=DEV).manual_seed(1000003 * seed + 17)


def _normal(g, shape, scale, dtype=torch.bfloat16):
    return torch.randn(shape, generator=g, device=DEV, dtype=torch.float32).mul_(scale).to(dtype)


def _gain(g, d):
    return 1.0 + 0.1 * torch.randn(d, generator=g, device=DEV)


def _weights(g, s):
    """Random weights as a checkpoint would hold them: N(0, 0.02^2) matrices, gains near one."""
    t = torch.bfloat16 if s.dtype == "bf16" else torch.float32
    d, F, hd, kvw = s.d_model, s.ffn_dim, s.n_heads * s.head_dim, s.n_kv_heads * s.head_dim
    layers = [dict(wq=_normal(g, (hd, d), 0.02, t), wk=_normal(g, (kvw, d), 0.02, t), wv=_normal(g, (kvw, d), 0.02, t),
                   wo=_normal(g, (d, hd), 0.02, t), wg=_normal(g, (F, d), 0.02, t), wu=_normal(g, (F, d), 0.02, t),
                   wd=_normal(g, (d, F), 0.02, t), attn_norm=_gain(g, d), mlp_norm=_gain(g, d))
              for _ in range(s.n_layers)]
    return dict(embed=_normal(g, (s.vocab, d), 0.02, t), final_norm=_gain(g, d), layers=layers)


def _inputs(case, seed):
    """The case's random values, the same for ``prepare`` and ``exact``."""
    s, n, g, path = _shape(case), lengths_of(case), _generator(seed), case["path"]
    L, k, t = int(n.sum()), int(n.size), torch.bfloat16 if s.dtype == "bf16" else torch.float32
    d, F, hd, kvw = s.d_model, s.ffn_dim, s.n_heads * s.head_dim, s.n_kv_heads * s.head_dim
    i = types.SimpleNamespace(s=s, n=n, L=L, k=k, t=t)
    if path in ("prefill", "decode"):
        i.weights, i.lm_head = _weights(g, s), _normal(g, (s.vocab, d), 0.02, t)
        m = L if path == "prefill" else k
        i.tokens = torch.randint(0, s.vocab, (m,), generator=g, device=DEV, dtype=torch.int32)
        if path == "decode":
            i.ctx_k, i.ctx_v = (_normal(g, (s.n_layers, L, kvw), 1.0, t) for _ in range(2))
            i.gen_k, i.gen_v = (_normal(g, (s.n_layers, k * N_NEW, kvw), 1.0, t) for _ in range(2))
    elif path in ("qkv", "mlp"):
        i.x, i.gain = _normal(g, (L, d), 1.0, torch.float32), _gain(g, d)
        if path == "qkv":
            i.w = _normal(g, (hd + 2 * kvw, d), 0.02)
        else:
            i.wg, i.wu, i.wd = _normal(g, (F, d), 0.02), _normal(g, (F, d), 0.02), _normal(g, (d, F), 0.02)
    elif path == "attention":
        i.q, i.kc, i.vc = _normal(g, (L, hd), 1.0), _normal(g, (L, kvw), 1.0), _normal(g, (L, kvw), 1.0)
    else:
        i.hidden, i.lm_head = _normal(g, (L, d), 1.0, torch.float32), _normal(g, (s.vocab, d), 0.02, t)
    return i


def _to_slots(a, plan):
    """Rows of the prompts' tokens, in original order, at their slots of the packed batch; zero pads."""
    kv = torch.from_numpy(plan.slot_kv.astype(np.int64)).to(a.device)
    return torch.where((kv >= 0)[:, None], a[kv.clamp_min(0)], torch.zeros((), dtype=a.dtype, device=a.device))


def prepare(case, seed):
    i, path = _inputs(case, seed), case["path"]
    s, st = i.s, types.SimpleNamespace(path=path)
    f32 = lambda *shape: torch.zeros(shape, dtype=torch.float32, device=DEV)      # noqa: E731
    half = lambda *shape: torch.zeros(shape, dtype=i.t, device=DEV)               # noqa: E731
    hd, kvw = s.n_heads * s.head_dim, s.n_kv_heads * s.head_dim
    if path == "decode":
        st.model = pp.DeviceModel(s, i.weights)
        st.gen = pp.Generation(st.model, types.SimpleNamespace(k_cache=i.ctx_k, v_cache=i.ctx_v), i.n, N_NEW)
        st.gen.gen_k.copy_(i.gen_k)
        st.gen.gen_v.copy_(i.gen_v)
        st.tokens, st.lm_head, st.logits = i.tokens, i.lm_head, f32(i.k, s.vocab)
        st.tokens_out = torch.zeros(i.k, dtype=torch.int32, device=DEV)
        rows = (s.n_layers, i.k, N_NEW, kvw)
        st.new_k, st.new_v = st.gen.gen_k.view(rows)[:, :, STEP], st.gen.gen_v.view(rows)[:, :, STEP]
        return st
    st.plan = pp.pp_pack(i.n, case["row"])
    st.dplan, st.cfg, st.eps = pp.DevicePlan(st.plan), pp.config_of(s), s.rms_eps
    T = st.plan.n_slots
    if path in ("prefill", "first_token"):
        st.lm_head, st.logits = i.lm_head, f32(i.k, s.vocab)
        st.first = torch.zeros(i.k, dtype=torch.int32, device=DEV)
        st.ft_ws = torch.empty(pp.pp_first_token_workspace_size(st.cfg, st.dplan), dtype=torch.uint8, device=DEV)
    if path == "prefill":
        st.model, st.tokens = pp.DeviceModel(s, i.weights), i.tokens
        st.prefill = pp.Prefill(st.model, st.dplan)
    elif path == "first_token":
        st.hidden = i.hidden
    elif path == "attention":
        st.ldq, st.kc, st.vc, st.q, st.out = hd, i.kc, i.vc, _to_slots(i.q, st.plan), half(T, hd)
    else:
        st.T, st.d, st.F, st.gain = T, s.d_model, s.ffn_dim, i.gain
        st.x, st.xn = _to_slots(i.x, st.plan), half(T, s.d_model)
        if path == "qkv":
            st.w, st.q, st.kc, st.vc = i.w, half(T, hd), half(i.L, kvw), half(i.L, kvw)
            st.table = torch.empty(st.plan.max_len * s.head_dim, dtype=torch.float32, device=DEV)
        else:
            st.w_gateup, st.w_down = pp.interleave_gate_up(i.wg, i.wu).contiguous(), i.wd
            st.act = half(T, s.ffn_dim)
    return st


# ----------------------------------------------------------------------------- one pass
def run(st):
    if st.path == "prefill":
        hidden, k, v = st.prefill(st.tokens)
        pp.pp_first_token(st.cfg, st.dplan, hidden, st.lm_head, st.ft_ws, st.first, st.logits)
        return {"hidden": hidden, "k": k, "v": v, "logits": st.logits}
    if st.path == "qkv":
        pp.pp_rmsnorm(pp.PP_BF16, st.x, st.gain, st.T, st.d, st.eps, st.xn)
        pp.pp_qkv_projection(st.cfg, st.dplan, st.xn, st.w, st.table, st.q, st.kc, st.vc)
        return {"q": st.q, "k": st.kc, "v": st.vc}
    if st.path == "mlp":   # x is the residual stream: each pass adds the MLP's output to it
        pp.pp_rmsnorm(pp.PP_BF16, st.x, st.gain, st.T, st.d, st.eps, st.xn)
        pp.pp_gemm(pp.PP_BF16, pp.PP_EPI_SWIGLU, st.xn, st.d, st.w_gateup, st.d, st.act, st.F, st.T, 2 * st.F, st.d,
                   st.dplan)
        pp.pp_gemm(pp.PP_BF16, pp.PP_EPI_RESIDUAL, st.act, st.F, st.w_down, st.F, st.x, st.d, st.T, st.d, st.F, st.dplan)
        return {"x": st.x, "act": st.act}
    if st.path == "attention":
        pp.pp_attention(st.cfg, st.dplan, st.q, st.ldq, st.kc, st.vc, st.out)
        return {"out": st.out}
    if st.path == "decode":
        st.gen.step(STEP, st.tokens, st.lm_head, st.tokens_out, st.logits)
        return {"k": st.new_k, "v": st.new_v, "logits": st.logits}
    pp.pp_first_token(st.cfg, st.dplan, st.hidden, st.lm_head, st.ft_ws, st.first, st.logits)
    return {"tokens": st.first, "logits": st.logits}


# ----------------------------------------------------------------------------- 64-bit results
def _norm(x, gain, eps):
    return x * torch.rsqrt(x.square().mean(-1, keepdim=True) + eps) * gain.double()


def _rope(x, pos, theta):
    D = x.shape[-1]
    a = pos.double()[:, None] * theta ** (-2.0 * torch.arange(D // 2, device=x.device, dtype=torch.float64) / D)
    c, s = a.cos()[:, None], a.sin()[:, None]
    lo, hi = x[..., : D // 2], x[..., D // 2:]
    return torch.cat([lo * c - hi * s, hi * c + lo * s], -1)


def _attend(q, k, v, causal):
    """q [nq, H, D] against k, v [nk, Hkv, D], one head at a time, in blocks of query rows."""
    out, R = torch.empty_like(q), q.shape[1] // k.shape[1]
    for h in range(q.shape[1]):
        kh, vh = k[:, h // R].contiguous(), v[:, h // R].contiguous()
        for a in range(0, q.shape[0], 4096):
            qb = q[a:a + 4096, h].contiguous()
            end = a + qb.shape[0] if causal else kh.shape[0]
            sc = qb @ kh[:end].t().contiguous() / math.sqrt(q.shape[2])
            if causal:
                rows = a + torch.arange(qb.shape[0], device=q.device)
                sc.masked_fill_(torch.arange(end, device=q.device)[None] > rows[:, None], -math.inf)
            out[a:a + 4096, h] = torch.softmax(sc, -1) @ vh[:end]
    return out


def _mlp(xn, wg, wu, wd):
    act = torch.nn.functional.silu(xn @ wg.double().t()) * (xn @ wu.double().t())
    return act, act @ wd.double().t()


def _segments(n):
    off = np.concatenate([[0], np.cumsum(n)])
    return [(int(a), int(b)) for a, b in zip(off[:-1], off[1:])]


def exact(case, seed):
    i, path = _inputs(case, seed), case["path"]
    s, n = i.s, i.n
    H, Hkv, D, eps = s.n_heads, s.n_kv_heads, s.head_dim, s.rms_eps
    spans = _segments(n)
    pos = torch.cat([torch.arange(int(l)) for l in n]).to(DEV)
    if path == "first_token":
        last = torch.tensor([b - 1 for _, b in spans], device=DEV)
        return {"tokens": None, "logits": i.hidden[last].to(i.t).double() @ i.lm_head.double().t()}
    if path == "attention":
        plan, out = pp.pp_pack(n, case["row"]), torch.zeros((i.L, H, D), dtype=torch.float64, device=DEV)
        for a, b in spans:
            out[a:b] = _attend(i.q[a:b].double().view(-1, H, D), i.kc[a:b].double().view(-1, Hkv, D),
                               i.vc[a:b].double().view(-1, Hkv, D), True)
        return {"out": _to_slots(out.view(i.L, H * D), plan)}
    if path in ("qkv", "mlp"):
        plan, x = pp.pp_pack(n, case["row"]), i.x.double()
        xn = _norm(x, i.gain, eps)
        if path == "mlp":
            act, y = _mlp(xn, i.wg, i.wu, i.wd)
            return {"x": _to_slots(x + y, plan), "act": _to_slots(act, plan)}
        q, k, v = (xn @ i.w.double().t()).split([H * D, Hkv * D, Hkv * D], -1)
        q, k = (_rope(a.reshape(i.L, -1, D), pos, s.rope_theta).reshape(i.L, -1) for a in (q, k))
        return {"q": _to_slots(q, plan), "k": k, "v": v}
    rows = i.tokens.long()
    x = i.weights["embed"][rows].double()
    m = x.shape[0]
    if path == "decode":
        pos = torch.from_numpy(n.astype(np.int64)).to(DEV) + STEP
    ks, vs = [], []
    for l, w in enumerate(i.weights["layers"]):
        xn = _norm(x, w["attn_norm"], eps)
        q = _rope((xn @ w["wq"].double().t()).view(m, H, D), pos, s.rope_theta)
        k = _rope((xn @ w["wk"].double().t()).view(m, Hkv, D), pos, s.rope_theta)
        v = (xn @ w["wv"].double().t()).view(m, Hkv, D)
        o = torch.empty_like(q)
        for p, (a, b) in enumerate(spans):
            if path == "prefill":
                o[a:b] = _attend(q[a:b], k[a:b], v[a:b], True)
            else:
                g0 = p * N_NEW
                kk, vv = (torch.cat([c[l, a:b].double(), g[l, g0:g0 + STEP].double(), new[p].reshape(1, -1)])
                          .view(-1, Hkv, D) for c, g, new in ((i.ctx_k, i.gen_k, k), (i.ctx_v, i.gen_v, v)))
                R = H // Hkv
                sc = (q[p].view(Hkv, R, 1, D) * kk.transpose(0, 1)[:, None]).sum(-1) / math.sqrt(D)
                o[p] = (torch.softmax(sc, -1)[..., None] * vv.transpose(0, 1)[:, None]).sum(2).view(H, D)
        x = x + o.reshape(m, H * D) @ w["wo"].double().t()
        x = x + _mlp(_norm(x, w["mlp_norm"], eps), w["wg"], w["wu"], w["wd"])[1]
        ks.append(k.reshape(m, -1))
        vs.append(v.reshape(m, -1))
    h = _norm(x, i.weights["final_norm"], eps)
    if path == "decode":
        return {"k": torch.stack(ks), "v": torch.stack(vs), "logits": h @ i.lm_head.double().t()}
    last = torch.tensor([b - 1 for _, b in spans], device=DEV)
    return {"hidden": h, "k": torch.stack(ks), "v": torch.stack(vs), "logits": h[last] @ i.lm_head.double().t()}
