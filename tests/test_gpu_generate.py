"""Greedy generation with packed KV caches on the GPU (section 4.8), through the C ABI,
against the generation oracle (full recomputation per token, section 2.2).

* float32 model: pp_generate's tokens equal the oracle's wherever the oracle's choice is
  clear (best logit ahead of the second by more than 1e-3; float32 errors are ~1e-6), and
  the generated cache rows meet the stated bar (2e-2 / 2e-3).
* bf16 models, teacher-forced (up to 16 prompts the projections stream the weights where that
  is the faster way, up to 256 they take the GEMM tiles with O and down in K splits, beyond
  that the prefill's GEMMs as they are): every pp_decode_step is fed the oracle's token, and the rows
  it appends to the cache and its logits are gated against the error of an ideal bf16
  pipeline (the oracle with every stored value rounded to bf16): max and mean error each
  <= 1.25x the floor's, as in the prefill's parity; its token must be the oracle's where the oracle's lead exceeds twice the logit error,
  else a valid argmax.
* the packed and the full-batching layouts give bit-identical tokens and generated rows,
  and pp_generate is bit-identical to the same steps taken one by one.
"""
import types

import numpy as np
import pytest
import torch

from oracle import decoder as D
from oracle import generate as G
from paper_2404_09529_amd import prepack as pp
from paper_2404_09529_amd import workloads as W

from .gpu_util import bf16_dev, f32_dev, gate_vs_floor, host64, i32_dev, oracle_weights, report, require_gpu

pytestmark = pytest.mark.gpu

BAR_MAX, BAR_MEAN = 2e-2, 2e-3


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    require_gpu()


def _prefill(case, lm_head):
    """GPU prefill (packed, bin size = longest prompt) and first token of every prompt."""
    model = pp.DeviceModel(case.shape, case.weights)
    dplan = pp.DevicePlan(pp.pp_pack(case.lengths, 0))
    pre = pp.Prefill(model, dplan)
    pre(i32_dev(case.tokens))
    lm = bf16_dev(lm_head) if case.shape.dtype == "bf16" else f32_dev(lm_head)
    ws = torch.empty(max(pp.pp_first_token_workspace_size(model.config, dplan), 1), dtype=torch.uint8,
                     device="cuda")
    first = torch.empty(len(case.lengths), dtype=torch.int32, device="cuda")
    pp.pp_first_token(model.config, dplan, pre.hidden, lm, ws, first)
    return model, pre, lm, first


def _prompts(case):
    off = np.concatenate([[0], np.cumsum(case.lengths)])
    return [case.tokens[off[i]:off[i + 1]] for i in range(len(case.lengths))]


def _gen_rows(gen, layer, i, n, which="k"):
    t = gen.gen_k if which == "k" else gen.gen_v
    r = int(gen.layout.gen_off[i])
    return host64(t[layer, r:r + n])


def _gap(logits):
    s = np.sort(logits)
    return s[-1] - s[-2]


# ----------------------------------------------------------------------------- float32: tokens and the bar
@pytest.mark.parametrize("lengths,n_new,n_layers", [
    ([5, 1, 17, 9, 40], 6, 2),
    ([1], 1, 1),                      # one prompt of one token, one step
    ([3] * 70, 3, 1),                 # more than 64 prompts (two LM-head prompt chunks)
    ([290, 30], 260, 1),              # over 256 context keys and over 256 generated keys
])
def test_fp32_generate_matches_oracle(lengths, n_new, n_layers):
    case = W.make_case(1, 3, n_layers=n_layers, lengths=lengths, random_gains=True)
    lm_head = W.draw_lm_head(case.wl, 3, case.shape)
    sh = D.Shape.of(case.shape)
    print(f"[generate] f32 lengths {lengths[:6]} (k={len(lengths)}) n_new {n_new}", flush=True)
    model, pre, lm, first = _prefill(case, lm_head)
    gen = pp.Generation(model, pre, case.lengths, n_new)
    toks = gen(first, lm)
    torch.cuda.synchronize()
    got = np.concatenate([first.cpu().numpy()[None], toks.cpu().numpy()]).T     # [k, 1 + n_new]
    picks = range(len(lengths)) if len(lengths) <= 8 else [0, 33, 69]
    w64, lm64 = oracle_weights(case.weights), lm_head.astype(np.float64)
    for i in picks:
        p = _prompts(case)[i]
        ref = G.generate(p, w64, sh, lm64, n_new + 1)
        f = G.teacher_forced(p, ref[:-1], w64, sh, lm64)
        gaps = [_gap(D.prefill_prompt(p, w64, sh).hidden[-1] @ lm64.T)] + [_gap(r) for r in f.logits]
        clear = next((t for t, g in enumerate(gaps) if g <= 1e-3), len(gaps))
        assert got[i][:clear].tolist() == ref[:clear].tolist(), (i, got[i].tolist(), ref.tolist())
        if clear == len(gaps):   # same tokens fed: the generated rows compare one to one
            for l in range(n_layers):
                for which, ref_rows in (("k", f.k[l]), ("v", f.v[l])):
                    mx, mean = report(f"f32 prompt {i} {which}{l}", _gen_rows(gen, l, i, n_new, which), ref_rows)
                    assert mx <= BAR_MAX and mean <= BAR_MEAN


# ----------------------------------------------------------------------------- bf16, teacher-forced
# a width past 4096 (the fused residual norm's 8-elements-per-thread form), 13B-like
WIDE = {"d5120": dict(d_model=5120, n_heads=40, n_kv_heads=40, ffn_dim=13824),
        # F = 5248 = 10 x 512 + 128: the down projection's last 1 KB segment holds 128 columns
        "f5248": dict(d_model=2048, n_heads=16, n_kv_heads=16, ffn_dim=5248),
        # a width the weight-streaming kernels do not take: GEMM tiles at any prompt count
        "d1024": dict(d_model=1024, n_heads=8, n_kv_heads=4, ffn_dim=2816),
        # H D < d: O's K is shorter than the row
        "h2": dict(d_model=1024, n_heads=2, n_kv_heads=2, ffn_dim=1024),
        # eight query heads per key/value head
        "r8": dict(d_model=2048, n_heads=16, n_kv_heads=2, ffn_dim=2816)}


def _bf16_case(model_name, lengths, n_layers, seed=0):
    if model_name in WIDE:
        dims = WIDE[model_name]
    else:
        s = W.MODELS[model_name]
        dims = dict(d_model=s.d_model, n_heads=s.n_heads, n_kv_heads=s.n_kv_heads, ffn_dim=s.ffn_dim)
    return W.make_case(6, seed, lengths=lengths, random_gains=True, n_layers=n_layers, **dims)


@pytest.mark.parametrize("model_name,lengths,n_layers,n_new", [
    ("llama-1.3b", [37, 1, 300, 5, 129], 2, 4),
    ("mistral-7b", [64, 260, 3], 1, 3),
    ("llama-1.3b", [3] * 62 + [40, 9, 300, 1, 2, 7, 5, 3], 1, 2),   # 70 prompts
    ("llama-1.3b", [5, 17, 2] * 6 + [130, 1], 1, 2),                 # 20 prompts, on the tiles
    ("mistral-7b", [4, 9, 1, 33] * 10, 1, 2),                        # 40 prompts, GQA
    ("llama-1.3b", [2, 11, 6, 1] * 16, 1, 2),                        # 64 prompts: one row tile
    ("mistral-7b", [3, 8, 1, 20] * 16, 1, 2),                        # 64 prompts, d 4096, GQA
    ("d5120", [37, 1, 300, 5], 1, 3),                                 # d 5120
    ("d5120", [4, 9, 1, 33] * 5, 1, 2),                               # d 5120, 20 prompts
    ("llama2-7b", [37, 1, 300, 5], 1, 3),                             # F 11008: down ends in half a 1 KB segment
    ("llama2-7b", [3] * 15 + [200], 1, 2),                            # 16 prompts: the 1 KB-segment kernels' limit
    ("f5248", [9, 130, 1], 1, 2),
])
def test_bf16_decode_steps_teacher_forced(model_name, lengths, n_layers, n_new):
    _teacher_forced(model_name, lengths, n_layers, n_new, range(len(lengths)))


def _teacher_forced(model_name, lengths, n_layers, n_new, picks):
    """Every step fed the oracle's tokens; the prompts in ``picks`` compared with the oracle."""
    case = _bf16_case(model_name, lengths, n_layers)
    lm_head = W.draw_lm_head(case.wl, 0, case.shape)
    sh = D.Shape.of(case.shape)
    k, V = len(lengths), case.shape.vocab
    print(f"[generate] bf16 {model_name} lengths {lengths} layers {n_layers} n_new {n_new}", flush=True)
    model, pre, lm, _ = _prefill(case, lm_head)
    gen = pp.Generation(model, pre, case.lengths, n_new)
    prompts = _prompts(case)
    w64, lm64 = oracle_weights(case.weights), lm_head.astype(np.float64)
    fed = np.random.default_rng(k).integers(0, V, (k, n_new + 1))   # prompts that are not compared: any tokens
    for i in picks:
        fed[i] = G.generate(prompts[i], w64, sh, lm64, n_new + 1)   # oracle's greedy
    ref = {i: G.teacher_forced(prompts[i], fed[i, :n_new], w64, sh, lm64) for i in picks}
    flo = {i: G.teacher_forced(prompts[i], fed[i, :n_new], w64, sh, lm64, rnd=D.round_bf16) for i in picks}
    rows = np.asarray(list(picks))
    logits = torch.empty((k, V), dtype=torch.float32, device="cuda")
    out = torch.empty(k, dtype=torch.int32, device="cuda")
    for t in range(n_new):
        gen.step(t, i32_dev(fed[:, t]), lm, out, logits)
        lg = host64(logits)
        tok = out.cpu().numpy()
        # the step's logits [picks, V] are one tensor of the gate
        want_t = np.stack([ref[i].logits[t] for i in picks])
        floor_t = np.stack([flo[i].logits[t] for i in picks])
        gate_vs_floor(f"{model_name} step {t} logits", [D.errors(lg[rows], want_t)], [D.errors(floor_t, want_t)])
        for i in picks:
            want = ref[i].logits[t]
            err = np.abs(lg[i] - want)
            slack = 2 * err.max()
            top = np.sort(want)[::-1]
            if top[0] - top[1] > slack:
                assert tok[i] == fed[i, t + 1], (t, i, tok[i], fed[i, t + 1])
            else:
                assert want[tok[i]] >= top[0] - slack
    for l in range(n_layers):
        for which in ("k", "v"):
            errs = []
            for i in picks:
                got = _gen_rows(gen, l, i, n_new, which)
                want = (ref[i].k if which == "k" else ref[i].v)[l]
                floor = (flo[i].k if which == "k" else flo[i].v)[l]
                (gm, ga), (fm, fa) = D.errors(got, want), D.errors(floor, want)
                errs.append((gm, ga, fm, fa))
            gm, ga = max(e[0] for e in errs), np.mean([e[1] for e in errs])
            fm, fa = max(e[2] for e in errs), np.mean([e[3] for e in errs])
            print(f"[parity] {model_name} generated {which}{l}: max {gm:.3e} mean {ga:.3e} "
                  f"(bf16 floor {fm:.3e} / {fa:.3e})", flush=True)
            gate_vs_floor(f"{model_name} generated {which}{l}", [(gm, ga)], [(fm, fa)])


# ----------------------------------------------------------------------------- layouts and entry points agree
@pytest.mark.parametrize("dims,lengths", [
    (dict(d_model=256, n_heads=2, n_kv_heads=2, ffn_dim=384), [5, 1, 300]),         # half a segment; a tail of 384
    (dict(d_model=512, n_heads=4, n_kv_heads=2, ffn_dim=768), [9] * 15 + [140]),    # one segment
    (dict(d_model=1024, n_heads=4, n_kv_heads=4, ffn_dim=1280), [9, 130, 1]),       # two
    (dict(d_model=512, n_heads=24, n_kv_heads=24, ffn_dim=512), [3, 40]),           # 24 O splits: three load batches in the norm
    (dict(d_model=768, n_heads=6, n_kv_heads=6, ffn_dim=896), [9, 130, 1]),         # O and down streamed only
    (dict(d_model=6144, n_heads=4, n_kv_heads=4, ffn_dim=640), [9, 130, 1, 4, 2]),  # O at its last prompt count there
    (dict(d_model=6144, n_heads=4, n_kv_heads=4, ffn_dim=640), [9, 130, 1, 4, 2, 3]),   # down only
    (dict(d_model=7168, n_heads=4, n_kv_heads=4, ffn_dim=640), [9, 130]),           # tiles only
])
def test_bf16_decode_steps_of_few_prompts(dims, lengths):
    """Up to 16 prompts: every choice between the streaming kernels and the tiles, two layers."""
    name = f"d{dims['d_model']}s h{dims['n_heads']}"
    WIDE[name] = dims
    _teacher_forced(name, lengths, 2, 2, sorted({0, 1, 2, len(lengths) - 1} & set(range(len(lengths)))))


@pytest.mark.parametrize("model_name,lengths,n_layers,n_new", [
    ("llama2-7b", [3] * 16 + [150], 1, 2),                            # 17 prompts: the first count on the tiles
    ("d1024", [9, 130, 1], 2, 3),
    ("d1024", [2, 5, 1] * 43, 1, 2),                                  # 129 prompts: partial sums over the chunks
    ("h2", [2, 1] * 33, 1, 2),
    ("d1024", [1, 2] * 128 + [1], 1, 2),                              # 257 prompts: the prefill's GEMMs as they are
])
def test_bf16_decode_steps_on_gemm_tiles(model_name, lengths, n_layers, n_new):
    test_bf16_decode_steps_teacher_forced(model_name, lengths, n_layers, n_new)


@pytest.mark.parametrize("model_name,lengths,n_layers,n_new", [
    # two layers: a layer's partial sums lie where the attention of the next writes its chunks
    ("d1024", [4, 9, 1, 33] * 5, 2, 2),
    ("d1024", [3, 1, 130] * 23, 2, 2),                                # 69 prompts
    ("d1024", [2, 5, 1] * 50, 2, 1),                                  # 150
    # the 128-row tiles of the split projections at real widths (O, down): 128 x 64 and 128 x 128
    ("llama2-7b", [2, 5, 1, 1, 3] * 14, 1, 1),                        # 70 prompts
    ("llama2-7b", [1, 2, 1] * 43, 1, 1),                              # 129: 128 x 128 and 128 x 256
    # eight query heads per key/value head: 10 prompts streamed, 20 on the tiles
    ("r8", [40, 1, 300, 9, 130] * 2, 1, 2),
    ("r8", [40, 1, 300, 9, 130] * 4, 1, 2),
])
def test_bf16_decode_steps_sampled(model_name, lengths, n_layers, n_new):
    """Larger steps: the prompts at the ends and around the row tiles' edges compared."""
    k = len(lengths)
    _teacher_forced(model_name, lengths, n_layers, n_new, sorted({0, 1, 2, 15, 31, 32, 63, 64, 127, 128, k - 1} & set(range(k))))


@pytest.mark.parametrize("model_name,lengths,n_layers,n_new", [
    ("llama-1.3b", [1, 300, 7, 129, 1, 64], 1, 5),
    ("mistral-7b", [700, 2, 33], 1, 5),
    ("d5120", [2, 150, 9], 1, 5),
    ("llama2-7b", [2, 150, 9, 1], 1, 5),
    # past 128 generated tokens: two chunks of generated keys per prompt (the packed layout's
    # attention work list against the full-batching layout's direct grid)
    ("llama-1.3b", [3, 260, 1, 40], 1, 140),
    # on the tiles: partial sums in K splits, 17 prompts and more
    ("d1024", [1, 140, 7, 2] * 5, 2, 4),
    ("d1024", [1, 140, 7, 2, 30] * 14, 2, 4),
    ("llama-1.3b", [2, 1, 9] * 43, 1, 3),
    ("r8", [3, 200, 1, 40], 2, 4),
])
def test_packed_and_padded_generation_are_bit_identical(model_name, lengths, n_layers, n_new):
    case = _bf16_case(model_name, lengths, n_layers, seed=1)
    lm_head = W.draw_lm_head(case.wl, 1, case.shape)
    model, pre, lm, first = _prefill(case, lm_head)
    packed = pp.Generation(model, pre, case.lengths, n_new)
    padded = pp.Generation(model, pre, case.lengths, n_new, padded=True)
    a = packed(first, lm).cpu().numpy()
    b = padded(first, lm).cpu().numpy()
    torch.cuda.synchronize()
    assert np.array_equal(a, b)
    for l in range(n_layers):
        for i in range(len(lengths)):
            for which in ("k", "v"):
                assert np.array_equal(_gen_rows(packed, l, i, n_new, which), _gen_rows(padded, l, i, n_new, which))
    # the full-batching cache is larger by the padding of every prompt to the longest
    assert padded.kv_cache_bytes() > packed.kv_cache_bytes()


@pytest.mark.parametrize("model_name,lengths,n_layers", [
    ("d1024", [3] * 70, 2),                                           # partial sums past 64 prompts
    ("llama-1.3b", [2, 1] * 65, 1),
    ("h2", [2, 1] * 40, 2),                                           # H D < d
    ("d1024", [3] * 20, 2),
    ("d1024", [3] * 10, 2),
])
def test_a_steps_bits_do_not_depend_on_room_or_on_other_prompts(model_name, lengths, n_layers):
    """Room for more generated tokens, or another prompt's length, changes no bit of a prompt's step."""
    def step(lens, n_new):
        case = _bf16_case(model_name, lens, n_layers, seed=3)
        lm_head = W.draw_lm_head(case.wl, 3, case.shape)
        case.tokens[:] = np.arange(case.tokens.size) % 97             # the same prompts whatever follows them
        model, pre, lm, _ = _prefill(case, lm_head)
        gen = pp.Generation(model, pre, case.lengths, n_new)
        k = len(lens)
        logits = torch.empty((k, case.shape.vocab), dtype=torch.float32, device="cuda")
        out = torch.empty(k, dtype=torch.int32, device="cuda")
        res = []
        for t in range(2):
            gen.step(t, i32_dev(np.arange(k) + 5 * t), lm, out, logits)
            res.append(logits.clone())
        torch.cuda.synchronize()
        return res + [torch.stack([gen.gen_k[l, int(r):int(r) + 2] for l in range(n_layers) for r in gen.layout.gen_off])]

    want = step(lengths, 2)
    assert bool(torch.isfinite(want[1]).all())
    for n_new in (129, 300):
        for a, b in zip(want, step(lengths, n_new)):
            assert torch.equal(a, b), n_new
    for a, b in zip(want[:2], step(lengths[:-1] + [400], 2)[:2]):
        assert torch.equal(a[:-1], b[:-1])


def test_scores_of_minus_infinity():
    """Keys whose score is -inf weigh nothing, and a row with no other key is not a number (the
    softmax of a row of -inf).  wk = -wq, so the step's own key is the negative of its query; a
    context of that key gives -|q|^2 = -inf everywhere, a key of zeros scores 0."""
    for k in (4, 20):                                                 # O merges the chunks; the tiles
        case = _bf16_case("llama-1.3b", [1, 5, 200, 300] * (k // 4), 1, seed=5)
        layer = case.weights["layers"][0]
        layer["wq"] = layer["wq"] * np.float32(1e22)
        layer["wk"] = -layer["wq"]
        lm = bf16_dev(W.draw_lm_head(case.wl, 5, case.shape))
        model = pp.DeviceModel(case.shape, case.weights)
        L, kvw = int(case.lengths.sum()), case.shape.n_kv_heads * case.shape.head_dim
        ctx_k = torch.zeros((1, L, kvw), dtype=torch.bfloat16, device="cuda")
        ctx_v = torch.ones_like(ctx_k)
        gen = pp.Generation(model, types.SimpleNamespace(k_cache=ctx_k, v_cache=ctx_v), case.lengths, 1)
        toks, out = i32_dev(np.arange(k) + 3), torch.empty(k, dtype=torch.int32, device="cuda")
        logits = torch.empty((k, case.shape.vocab), dtype=torch.float32, device="cuda")
        gen.step(0, toks, lm, out, logits)                            # the step's keys
        off = gen.layout.ctx_off
        for i in range(k):
            ctx_k[0, off[i]:off[i] + int(case.lengths[i])] = gen.gen_k[0, i]
        ctx_k[0, off[3] + 150] = 0                                    # prompt 3: one key of score 0
        gen.step(0, toks, lm, out, logits)
        torch.cuda.synchronize()
        nan = torch.isnan(logits).all(1).cpu().numpy()
        assert nan.tolist() == [i != 3 for i in range(k)], (k, nan)
        assert bool(torch.isfinite(logits[3]).all()) and out.cpu().tolist()[:3] == [-1, -1, -1]


def test_generate_equals_steps_one_by_one():
    case = _bf16_case("llama-1.3b", [9, 200, 1], 2, seed=2)
    lm_head = W.draw_lm_head(case.wl, 2, case.shape)
    n_new = 4
    model, pre, lm, first = _prefill(case, lm_head)
    whole = pp.Generation(model, pre, case.lengths, n_new)
    toks = whole(first, lm).clone()
    steps = pp.Generation(model, pre, case.lengths, n_new)
    prev = first
    outs = []
    for t in range(n_new):
        out = torch.empty_like(first)
        steps.step(t, prev, lm, out)
        outs.append(out)
        prev = out
    torch.cuda.synchronize()
    assert np.array_equal(toks.cpu().numpy(), torch.stack(outs).cpu().numpy())
    for l in range(2):
        assert torch.equal(whole.gen_k[l], steps.gen_k[l]) and torch.equal(whole.gen_v[l], steps.gen_v[l])


def test_graph_replays_match_eager_generation():
    """The whole generation captured as one HIP graph: every replay, with eager work and
    synchronisations between replays, gives the eager call's tokens and generated rows."""
    case = _bf16_case("llama-1.3b", [11, 1, 130, 4], 2, seed=4)
    lm_head = W.draw_lm_head(case.wl, 4, case.shape)
    model, pre, lm, first = _prefill(case, lm_head)
    eager = pp.Generation(model, pre, case.lengths, 6)
    want = eager(first, lm).clone()
    torch.cuda.synchronize()
    g = pp.Generation(model, pre, case.lengths, 6)
    g.capture(first, lm)
    for rep in range(3):
        g.gen_k.zero_()
        g.tokens.fill_(-5)
        torch.cuda.synchronize()
        got = g.replay()
        torch.cuda.synchronize()
        assert torch.equal(got, want), rep
        assert torch.equal(g.gen_k, eager.gen_k) and torch.equal(g.gen_v, eager.gen_v), rep
        eager(first, lm)                       # eager work between replays
        torch.cuda.synchronize()
