// Generation with packed KV caches (section 4.8): the cache layouts and the decode step.
//
// Host side only.  pp_gen_layout_make places every prompt's keys and values (packed: the
// prefill's per-prompt cache plus n_new rows per prompt; full batching: k rows of
// m + n_new slots).  pp_decode_step validates everything, carves the caller's workspace and
// enqueues, without host synchronisation:
//
//   start: positions, RoPE rows, append rows; embedding of the k fed tokens and the first norm
//   per layer: rmsnorm -> QKV projection with RoPE and the append to the generation cache
//              (the prefill's fused epilogue) ->
//              split-key decode attention + combine -> O GEMM (+residual) -> rmsnorm ->
//              gate/up GEMM with SwiGLU -> down GEMM (+residual); with the split-K GEMMs
//              the residual adds of O and down happen in the norm that follows each
//   final rmsnorm -> LM head and greedy choice (the first-token kernels, one row per prompt).
// The projections: for bf16 steps of up to 16 prompts, weight-streaming GEMMs for one row
// per prompt at the widths where they are faster (QKV and gate/up with their epilogues in the
// kernel; O and down as split-K partial sums that the next norm adds); up to 256 prompts the
// prefill's GEMM tiles, O and down split likewise; otherwise the prefill's GEMM kernels with M = k.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "kernels.h"
#include "prepack.h"
#include "status.h"

namespace {

constexpr size_t kAlign = 256;
size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }
size_t elem_size(int dtype) { return dtype == PP_BF16 ? 2 : 4; }

struct Layout {
    size_t x = 0, xn = 0, q = 0, attn = 0, act = 0, part = 0, table = 0, ints = 0, ft = 0, gpart = 0,
           total = 0;
};

// The projections of a decode step as (N, K).
struct Proj {
    int N, K;
};
void projections(const pp_config* c, Proj (&p)[4]) {
    const int d = c->d_model, hd = c->n_heads * c->head_dim;
    p[0] = {(c->n_heads + 2 * c->n_kv_heads) * c->head_dim, d};   // QKV
    p[1] = {d, hd};                                               // O
    p[2] = {2 * c->ffn_dim, d};                                   // gate/up
    p[3] = {d, c->ffn_dim};                                       // down
}

// bf16 widths whose O and down projections may leave partial sums to the residual norm.
bool split_width(const pp_config* c) { return c->dtype == PP_BF16 && ppk::residual_rmsnorm_ok(c->d_model); }

// How a step's projections run.  Up to 16 prompts take the weight-streaming kernels of k_decode.hip
// where those are the faster ones, projection by projection; up to 256 the prefill's GEMM tiles, O
// and down in K splits; more, and widths that the residual norm does not take, the prefill's GEMMs
// as they are.
// From 17 prompts on the weights are no longer nearly all that a projection reads: the streaming
// kernels' wavefronts each fetch every prompt's row, and O's workgroups each merge every prompt's
// attention chunks.  At 48 prompts of a grouped-query 7B layer they took 23 / 30 / 90 / 50 us (QKV, O,
// gate/up, down) against 19 / 5 + 12 / 52 / 28 for the tiles (O with its chunk merge as a kernel of its own).
struct Plan {
    bool split;    // O and down leave partial sums to the norm that follows
    bool paired;   // QKV and gate/up streamed
    bool o;        // O streamed, merging the attention's chunks
    bool down;     // down streamed
};
constexpr int kSplitPrompts = 256;
Plan plan_of(const pp_config* c, int k) {
    const int d = c->d_model;
    Plan p{split_width(c) && k <= kSplitPrompts, false, false, false};
    if (!p.split || k > 16) return p;
    // QKV and gate/up where a row is a power of two of the 512-column segments (or half a one): a
    // step of two layers at d 512 on the tiles 82 us, streamed 71; d 1024: 109 and 102.
    // O and down, the same step with both on the tiles, down streamed, O streamed, both streamed (QKV
    // and gate/up on the tiles): d 1024, 1 prompt: 126, 121, 114, 109 us; d 3072: 240, 227, 224, 212;
    // d 5120: 413, 400, 402, 387, and at 16 prompts, every one of which each of O's workgroups
    // merges, 438, 434, 448, 446; d 6144: 522, 489, 518, 483, and at 10 prompts 536, 503, 546, 509;
    // d 8192, one layer: 471, 475, 475, 477.
    p.paired = ppk::decode_paired_ok(d);
    p.o = d <= 4096 || (d <= 6144 && k * d <= 32768);
    p.down = d <= 6144;
    return p;
}

// The K splits that the tiles may take for O and down: 16 up to 128 prompts, fewer for more (2048 rows
// of partial sums in all; few shapes would take more).  A function of k alone, so
// that a prompt's results depend neither on the room reserved for generated tokens nor on the
// lengths of the other prompts.
int tile_splits(int k) { return std::min(16, 2048 / k); }

int chunks(int n) { return (n + ppk::kDecodeChunk - 1) / ppk::kDecodeChunk; }

Layout layout_of(const pp_config* c, const pp_gen_dlayout* g) {
    const size_t k = g->k, e = elem_size(c->dtype);
    const size_t d = c->d_model, F = c->ffn_dim, D = c->head_dim;
    const size_t qkv_w = size_t(c->n_heads + 2 * c->n_kv_heads) * D, hd = size_t(c->n_heads) * D;
    const size_t nch = size_t(chunks(g->max_len) + chunks(g->n_new));
    Layout L;
    size_t off = 0;
    auto take = [&](size_t bytes) {
        const size_t at = off;
        off += align_up(bytes);
        return at;
    };
    L.x = take(k * d * 4);
    L.xn = take(k * d * e);
    L.q = take(c->dtype == PP_BF16 ? k * hd * 2 : k * qkv_w * 4);   // bf16: rotated queries only
    L.attn = take(k * hd * e);
    L.act = take(k * F * e);
    const Plan plan = plan_of(c, g->k);
    size_t sums = 0;   // bytes of O's and down's partial sums
    if (plan.split) {
        Proj p[4];
        projections(c, p);
        int splits = plan.o && plan.down ? 0 : tile_splits(g->k);
        if (plan.o) splits = std::max(splits, ppk::skinny_split(p[1].N, p[1].K).splits);
        if (plan.down) splits = std::max(splits, ppk::decode_gemm_splits(g->k, p[3].N, p[3].K));
        sums = size_t(splits) * k * d * 4;
    }
    // A streamed O merges the attention's chunk results while it leaves its sums, which have a region
    // of their own; else the chunk results are merged before, and the sums take their place and that of
    // a region of k d floats which the size of a workspace has always held.
    L.gpart = take(k * d * 4);
    L.part = take(k * size_t(c->n_heads) * nch * (D + 4) * 4);
    if (plan.o) L.gpart = take(sums);
    else if (sums > off - L.gpart) take(sums - (off - L.gpart));
    L.table = take(k * (D / 2) * sizeof(float2));
    L.ints = take((4 * k + 1) * sizeof(int32_t));
    L.ft = take(ppk::first_token_workspace(c->dtype, g->k, c->vocab, c->d_model));
    L.total = off;
    return L;
}

pp_status validate_layout(const pp_config* c, const pp_gen_dlayout* g) {
    if (!g) return pp::fail(PP_ERR_INVALID_ARG, "layout is NULL");
    if (g->k <= 0 || g->n_new <= 0 || g->max_len <= 0 || (g->padded != 0 && g->padded != 1))
        return pp::fail(PP_ERR_INVALID_ARG, "layout k %d, n_new %d, max_len %d, padded %d", g->k, g->n_new,
                        g->max_len, g->padded);
    if (g->ctx_rows <= 0 || g->gen_rows < int64_t(g->k) * g->n_new || g->ctx_rows > INT32_MAX ||
        g->gen_rows > INT32_MAX)
        return pp::fail(PP_ERR_INVALID_ARG, "layout rows: ctx %lld, gen %lld", (long long)g->ctx_rows,
                        (long long)g->gen_rows);
    if (!g->ctx_off || !g->ctx_span || !g->ctx_valid || !g->pos0 || !g->gen_off)
        return pp::fail(PP_ERR_INVALID_ARG, "a device layout array is NULL");
    const int R = c->n_heads / c->n_kv_heads;
    if (R != 1 && R != 2 && R != 4 && R != 8)
        return pp::fail(PP_ERR_UNSUPPORTED, "decode attention needs n_heads / n_kv_heads in {1, 2, 4, 8} (%d)", R);
    return PP_OK;
}

pp_status check_buffers(const pp_config* c, const pp_gen_dlayout* g, const void* lm_head, const void* ctx_k,
                        const void* ctx_v, const void* gen_k, const void* gen_v, const void* workspace,
                        size_t workspace_bytes) {
    if (!lm_head || !ctx_k || !ctx_v || !gen_k || !gen_v)
        return pp::fail(PP_ERR_INVALID_ARG, "lm_head and the four caches must be non-NULL");
    if (!workspace) return pp::fail(PP_ERR_INVALID_ARG, "workspace is NULL");
    if (reinterpret_cast<uintptr_t>(workspace) % kAlign)
        return pp::fail(PP_ERR_INVALID_ARG, "workspace is not %zu-byte aligned", kAlign);
    const size_t need = layout_of(c, g).total;
    if (workspace_bytes < need)
        return pp::fail(PP_ERR_BUFFER_TOO_SMALL, "workspace of %zu bytes < %zu needed", workspace_bytes, need);
    return PP_OK;
}

pp_status check_all(const pp_config* cfg, const pp_weights* w, const pp_gen_dlayout* g) {
    if (pp_status st = pp::validate_config(cfg)) return st;
    if (pp_status st = pp::validate_weights(cfg, w)) return st;
    return validate_layout(cfg, g);
}

// Enqueue one decode step (arguments already validated).
void enqueue_step(const pp_config* cfg, const pp_weights* w, const pp_gen_dlayout* g, int step,
                  const int32_t* tokens_in, const void* lm_head, const void* ctx_k, const void* ctx_v, void* gen_k,
                  void* gen_v, void* workspace, float* logits, int32_t* tokens_out, hipStream_t s) {
    const Layout L = layout_of(cfg, g);
    const int dt = cfg->dtype;
    const bool bf = dt == PP_BF16;
    const int k = g->k;
    const int d = cfg->d_model, H = cfg->n_heads, Hkv = cfg->n_kv_heads, D = cfg->head_dim, F = cfg->ffn_dim;
    const int qkv_w = (H + 2 * Hkv) * D, hd = H * D, kvw = Hkv * D;
    const float eps = cfg->rms_eps;
    const size_t e = elem_size(dt);

    char* ws = static_cast<char*>(workspace);
    float* x = reinterpret_cast<float*>(ws + L.x);
    void* xn = ws + L.xn;
    void* q = ws + L.q;
    void* attn = ws + L.attn;
    void* act = ws + L.act;
    float* part = reinterpret_cast<float*>(ws + L.part);
    float2* table = reinterpret_cast<float2*>(ws + L.table);
    int32_t* slot_pos = reinterpret_cast<int32_t*>(ws + L.ints);
    int32_t* slot_kv = slot_pos + k;
    const size_t ctx_layer = size_t(g->ctx_rows) * kvw * e, gen_layer = size_t(g->gen_rows) * kvw * e;
    // the prompts' context chunks together: at most ceil(ctx_rows / chunk) + k, as every prompt's
    // span lies in its own ctx_rows (and at most k x the longest prompt's)
    const int n_ctx_items = static_cast<int>(std::min<int64_t>(int64_t(k) * chunks(g->max_len),
                                                               (g->ctx_rows + ppk::kDecodeChunk - 1) / ppk::kDecodeChunk + k));
    const ppk::DecodeLayout Ly{k, chunks(g->max_len), chunks(g->n_new), n_ctx_items, g->ctx_off, g->ctx_span,
                               g->ctx_valid, g->pos0, g->gen_off};
    const Plan plan = plan_of(cfg, k);
    const int splits = tile_splits(k);
    float* gpart = reinterpret_cast<float*>(ws + L.gpart);

    // the split-K residual projections (O, down) leave their partial sums in gpart; the next
    // norm adds them to x (pending = their split count) before normalising
    int pending = 0;
    auto norm = [&](const float* gain, void* out) {
        if (plan.split)
            ppk::residual_rmsnorm(x, gpart, pending, k, d, gain, out, eps, s);
        else
            ppk::rmsnorm(dt, x, gain, out, k, d, eps, s);
        pending = 0;
    };
    ppk::decode_start(dt, Ly, step, D, cfg->rope_theta, table, slot_pos, slot_kv, x, w->embed, cfg->vocab,
                      tokens_in, d, w->attn_norm[0], xn, eps, s);
    for (int l = 0; l < cfg->n_layers; ++l) {
        const void* ck = static_cast<const char*>(ctx_k) + l * ctx_layer;
        const void* cv = static_cast<const char*>(ctx_v) + l * ctx_layer;
        void* gk = static_cast<char*>(gen_k) + l * gen_layer;
        void* gv = static_cast<char*>(gen_v) + l * gen_layer;
        if (l > 0) norm(w->attn_norm[l], xn);
        if (bf) {
            const ppk::QkvOut qo{q, hd, gk, gv, kvw, table, slot_pos, slot_kv, H, Hkv};
            if (plan.paired)
                ppk::decode_gemm(ppk::kQkvRope, xn, d, k, w->wqkv[l], d, qkv_w, d, gpart,
                                 ppk::DecodeEpi{nullptr, 0, qo}, s);
            else
                ppk::qkv_rope_bf16(xn, d, w->wqkv[l], d, k, d, nullptr, 0, qo, s);
            ppk::decode_attention(dt, q, hd, ck, cv, gk, gv, kvw, Ly, step, H, Hkv, D, part, plan.o ? nullptr : attn, hd, s);
            if (plan.o) {
                const ppk::AttnChunks ac{part, g->ctx_span, step, Ly.n_ctx_chunks, Ly.n_ctx_chunks + Ly.n_gen_chunks, H};
                ppk::decode_gemm_o(k, ac, w->wo[l], hd, d, hd, gpart, s);
                pending = ppk::skinny_split(d, hd).splits;
            } else if (plan.split) {
                ppk::gemm_partial_bf16(attn, hd, w->wo[l], hd, gpart, k, d, hd, splits, s);
                pending = ppk::gemm_partial_splits(k, d, hd, splits);
            } else {
                ppk::gemm_bf16(ppk::kResidual, attn, hd, w->wo[l], hd, x, d, k, d, hd, nullptr, 0, s);
            }
        } else {
            const ppk::QkvOut qo{q, qkv_w, gk, gv, kvw, table, slot_pos, slot_kv, H, Hkv};
            ppk::qkv_rope_f32(static_cast<const float*>(xn), d, static_cast<const float*>(w->wqkv[l]), d, k, d, D, qo, s);
            ppk::decode_attention(dt, q, qkv_w, ck, cv, gk, gv, kvw, Ly, step, H, Hkv, D, part, attn, hd, s);
            ppk::gemm_f32(ppk::kResidual, static_cast<const float*>(attn), hd, static_cast<const float*>(w->wo[l]),
                          hd, x, d, k, d, hd, s);
        }
        norm(w->mlp_norm[l], xn);
        if (bf) {
            if (plan.paired)
                ppk::decode_gemm(ppk::kSwiGLU, xn, d, k, w->w_gateup[l], d, 2 * F, d, gpart,
                                 ppk::DecodeEpi{act, F, ppk::QkvOut{}}, s);
            else
                ppk::gemm_bf16(ppk::kSwiGLU, xn, d, w->w_gateup[l], d, act, F, k, 2 * F, d, nullptr, 0, s);
            if (plan.down) {
                ppk::decode_gemm(ppk::kResidual, act, F, k, w->w_down[l], F, d, F, gpart, ppk::DecodeEpi{}, s);
                pending = ppk::decode_gemm_splits(k, d, F);
            } else if (plan.split) {
                ppk::gemm_partial_bf16(act, F, w->w_down[l], F, gpart, k, d, F, splits, s);
                pending = ppk::gemm_partial_splits(k, d, F, splits);
            } else {
                ppk::gemm_bf16(ppk::kResidual, act, F, w->w_down[l], F, x, d, k, d, F, nullptr, 0, s);
            }
        } else {
            ppk::gemm_f32(ppk::kSwiGLU, static_cast<const float*>(xn), d, static_cast<const float*>(w->w_gateup[l]), d,
                          static_cast<float*>(act), F, k, 2 * F, d, s);
            ppk::gemm_f32(ppk::kResidual, static_cast<const float*>(act), F, static_cast<const float*>(w->w_down[l]),
                          F, x, d, k, d, F, s);
        }
    }
    // the final norm's rows go straight to where the LM head reads them, in its type: a gather of
    // them from float32, with the same rounding, was a launch of 4.7 us
    norm(w->final_norm, ws + L.ft);
    ppk::next_token(dt, k, lm_head, cfg->vocab, d, ws + L.ft, logits, tokens_out, s);
}

}  // namespace

extern "C" pp_status pp_gen_layout_make(const int32_t* lengths, int32_t k, int32_t n_new, int32_t padded,
                                        pp_gen_layout* layout) {
    pp::clear_error();
    if (!lengths || !layout) return pp::fail(PP_ERR_INVALID_ARG, "lengths and layout must be non-NULL");
    if (k <= 0 || n_new <= 0 || (padded != 0 && padded != 1))
        return pp::fail(PP_ERR_INVALID_ARG, "k %d, n_new %d, padded %d", k, n_new, padded);
    if (!layout->ctx_off || !layout->ctx_span || !layout->ctx_valid || !layout->pos0 || !layout->gen_off)
        return pp::fail(PP_ERR_INVALID_ARG, "a layout array is NULL");
    int64_t total = 0;
    int32_t m = 0;
    for (int32_t i = 0; i < k; ++i) {
        if (lengths[i] <= 0) return pp::fail(PP_ERR_INVALID_ARG, "length %d of prompt %d", lengths[i], i);
        total += lengths[i];
        m = std::max(m, lengths[i]);
    }
    const int64_t row = int64_t(m) + n_new;
    const int64_t ctx_rows = padded ? int64_t(k) * row : total;
    const int64_t gen_rows = padded ? int64_t(k) * row : int64_t(k) * n_new;
    if (ctx_rows > INT32_MAX || gen_rows > INT32_MAX)
        return pp::fail(PP_ERR_INVALID_ARG, "%lld cache rows exceed the int32 row index", (long long)gen_rows);
    int64_t off = 0;
    for (int32_t i = 0; i < k; ++i) {
        layout->ctx_off[i] = static_cast<int32_t>(padded ? int64_t(i) * row : off);
        layout->ctx_span[i] = padded ? m : lengths[i];
        layout->ctx_valid[i] = lengths[i];
        layout->pos0[i] = lengths[i];
        layout->gen_off[i] = static_cast<int32_t>(padded ? int64_t(i) * row + m : int64_t(i) * n_new);
        off += lengths[i];
    }
    layout->k = k;
    layout->n_new = n_new;
    layout->padded = padded;
    layout->max_len = m;
    layout->ctx_rows = ctx_rows;
    layout->gen_rows = gen_rows;
    return PP_OK;
}

extern "C" pp_status pp_decode_workspace_size(const pp_config* cfg, const pp_gen_dlayout* layout, size_t* bytes) {
    pp::clear_error();
    if (pp_status st = pp::validate_config(cfg)) return st;
    if (pp_status st = validate_layout(cfg, layout)) return st;
    if (!bytes) return pp::fail(PP_ERR_INVALID_ARG, "bytes is NULL");
    *bytes = layout_of(cfg, layout).total;
    return PP_OK;
}

extern "C" pp_status pp_decode_step(const pp_config* cfg, const pp_weights* w, const pp_gen_dlayout* layout,
                                    int32_t step, const int32_t* tokens_in, const void* lm_head, const void* ctx_k,
                                    const void* ctx_v, void* gen_k, void* gen_v, void* workspace,
                                    size_t workspace_bytes, float* logits, int32_t* tokens_out, void* stream) {
    pp::clear_error();
    if (pp_status st = check_all(cfg, w, layout)) return st;
    if (step < 0 || step >= layout->n_new)
        return pp::fail(PP_ERR_INVALID_ARG, "step %d outside [0, n_new = %d)", step, layout->n_new);
    if (!tokens_in || !tokens_out) return pp::fail(PP_ERR_INVALID_ARG, "tokens_in and tokens_out must be non-NULL");
    if (pp_status st = check_buffers(cfg, layout, lm_head, ctx_k, ctx_v, gen_k, gen_v, workspace, workspace_bytes))
        return st;
    (void)hipGetLastError();
    enqueue_step(cfg, w, layout, step, tokens_in, lm_head, ctx_k, ctx_v, gen_k, gen_v, workspace, logits, tokens_out,
                 static_cast<hipStream_t>(stream));
    const hipError_t err = hipGetLastError();
    if (err != hipSuccess) return pp::fail(PP_ERR_HIP, "decode step launch failed: %s", hipGetErrorString(err));
    return PP_OK;
}

extern "C" pp_status pp_generate(const pp_config* cfg, const pp_weights* w, const pp_gen_dlayout* layout,
                                 int32_t n_steps, const int32_t* tokens_first, const void* lm_head, const void* ctx_k,
                                 const void* ctx_v, void* gen_k, void* gen_v, void* workspace,
                                 size_t workspace_bytes, int32_t* tokens, void* stream) {
    pp::clear_error();
    if (pp_status st = check_all(cfg, w, layout)) return st;
    if (n_steps < 0 || n_steps > layout->n_new)
        return pp::fail(PP_ERR_INVALID_ARG, "n_steps %d outside [0, n_new = %d]", n_steps, layout->n_new);
    if (n_steps == 0) return PP_OK;
    if (!tokens_first || !tokens) return pp::fail(PP_ERR_INVALID_ARG, "tokens_first and tokens must be non-NULL");
    if (pp_status st = check_buffers(cfg, layout, lm_head, ctx_k, ctx_v, gen_k, gen_v, workspace, workspace_bytes))
        return st;
    (void)hipGetLastError();
    hipStream_t s = static_cast<hipStream_t>(stream);
    const int k = layout->k;
    for (int t = 0; t < n_steps; ++t)
        enqueue_step(cfg, w, layout, t, t == 0 ? tokens_first : tokens + int64_t(t - 1) * k, lm_head, ctx_k, ctx_v,
                     gen_k, gen_v, workspace, nullptr, tokens + int64_t(t) * k, s);
    const hipError_t err = hipGetLastError();
    if (err != hipSuccess) return pp::fail(PP_ERR_HIP, "generate launch failed: %s", hipGetErrorString(err));
    return PP_OK;
}
