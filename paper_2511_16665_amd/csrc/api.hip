// C ABI of libtlt (see include/tlt.h): argument validation, workspace carving, and the sequence of
// kernel launches that makes up each of the four calls of the speculative-decoding step.
#include "../../include/tlt.h"

#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstring>
#include <functional>
#include <map>
#include <new>
#include <vector>

#include "kernels.h"

using namespace tlt;

namespace {

enum { CLS_GEMM = 0, CLS_ATTN = 1, CLS_COMMIT = 2, CLS_OTHER = 3, CLS_GEMM_DRAFT = 4, CLS_ATTN_DRAFT = 5, CLS_N = 6 };

struct ProfRec {
    int cls;
    double flops, bytes;
};

struct Plan {  // byte offsets into the workspace
    size_t x, xn, qkv, rope_cs, rope_at, parts, att, g, u, act, logits, argmax, feat, pool_token, pool_score, pool_parent,
        pool_depth, pool_mask, fr_token, fr_src, fr_pool, fr_mask, attn_ws, accept_ws, topk_ws, status, total;
    size_t attn_ws_bytes, parts_bytes;
    int max_rows, pool_cap, feat_rows;
};

size_t align_up(size_t v) { return (v + 255) & ~(size_t)255; }

constexpr int kMaxProvisionalRows = 128;   // rows of one expansion past the committed drafter entries (two mask words)

bool plan_workspace(const tlt_model_cfg& c, int B, int n, int D, int K, int max_ctx, Plan& p) {
    if (B < 1 || n < 1 || n > TLT_MAX_TREE || D < 0 || D > TLT_MAX_DEPTH || K < 1 || K > TLT_MAX_TOPK || max_ctx < 1)
        return false;
    const size_t esz = c.dtype == TLT_F32 ? 4 : 2;
    const size_t R = (size_t)B * std::max(n, K);
    const size_t h = c.hidden, F = c.mlp, V = c.vocab;
    const size_t qkv_dim = (size_t)(c.n_q_heads + 2 * c.n_kv_heads) * c.head_dim;
    p.max_rows = (int)R;
    p.pool_cap = K + std::max(0, D - 1) * K * K;
    // feature rows per sequence: the root's + one per drafter row of an expansion (deterministic:
    // K per level after the first; sampled: one per template node with children, fewer than n)
    p.feat_rows = std::max(1 + std::max(0, D - 1) * K, n);
    size_t o = 0;
    auto take = [&](size_t bytes) {
        size_t at = o;
        o = align_up(o + bytes);
        return at;
    };
    p.x = take(R * h * 4);
    p.xn = take(R * 2 * h * esz);
    p.qkv = take(R * qkv_dim * esz);
    // cosines, sines and cache slots of a forward's rows: written by its first layer, read by the others
    p.rope_cs = take(R * (size_t)c.head_dim * 4);
    p.rope_at = take(R * 8);
    // fp32 partial products of the projections whose sum joins the fp32 residual stream (or feeds the rotary kernel)
    // (room for four slices of the widest product at the largest row count; a plan with more cuts than fit is not taken)
    p.parts_bytes = std::max(c.dtype == TLT_BF16 ? gemm_parts_max_bytes() : (size_t)0, (c.dtype == TLT_BF16 ? 4 : 1) * R * std::max(h, qkv_dim) * 4);
    p.parts = take(p.parts_bytes);
    p.att = take(R * (size_t)c.n_q_heads * c.head_dim * esz);
    p.g = take(R * F * esz);
    p.u = take(R * F * esz);
    p.act = take(R * F * esz);
    p.logits = take(R * V * 4);
    p.argmax = take(R * 4);
    p.feat = take((size_t)B * p.feat_rows * h * 4);
    p.pool_token = take((size_t)B * p.pool_cap * 4);
    p.pool_score = take((size_t)B * p.pool_cap * 4);
    p.pool_parent = take((size_t)B * p.pool_cap * 4);
    p.pool_depth = take((size_t)B * p.pool_cap * 4);
    p.pool_mask = take((size_t)B * p.pool_cap * 16);
    const size_t FRN = (size_t)B * std::max(n, K);   // rows of one drafter pass
    p.fr_token = take(FRN * 4);
    p.fr_src = take(FRN * 4);
    p.fr_pool = take(FRN * 4);
    p.fr_mask = take(FRN * 16);
    p.attn_ws_bytes = attention_workspace_bytes(B, std::max(n, K), c.n_q_heads, c.n_kv_heads, c.head_dim, max_ctx);
    p.attn_ws = take(p.attn_ws_bytes);
    p.accept_ws = take(accept_sample_workspace_bytes(B, c.vocab));
    p.topk_ws = take(row_topk_workspace_bytes(B * K, c.vocab, K));
    p.status = take(256);   // device-side status word (see tlt_device_status)
    p.total = o;
    return true;
}

bool cfg_ok(const tlt_model_cfg* c) {
    if (!c) return false;
    if (c->n_layers < 1 || c->hidden < 4 || c->hidden % 4 || c->n_q_heads < 1 || c->n_kv_heads < 1 ||
        c->n_q_heads % c->n_kv_heads || c->head_dim < 64 || c->head_dim % 64 || c->head_dim > 256 || c->mlp < 1 ||
        c->vocab < 1 || c->page_size < 1 || !(c->rms_eps > 0.f) || !(c->rope_theta > 0.f))
        return false;
    if (c->dtype != TLT_F32 && c->dtype != TLT_BF16) return false;
    // 16-byte row chunks in the cache and the activations
    const int esz = c->dtype == TLT_F32 ? 4 : 2;
    if ((c->head_dim * esz) % 16) return false;
    return true;
}

}  // namespace

struct tlt_ctx {
    tlt_model_cfg cfg;
    tlt_weights target, draft;
    std::vector<tlt_layer_weights> target_layers, draft_layers;
    bool have_draft = false;
    int max_batch, max_n, max_depth, max_topk, max_ctx;
    char* ws = nullptr;
    Plan plan;
    int hip_error = 0;
    int attn_impl = -1;  // -1: pick by dtype/shape
    bool oproj_f32 = true;   // the output projection's product reaches the residual stream unrounded
    // partial products in the workspace that the residual stream x has not absorbed yet: x (+)= their sum, formed
    // by the next kernel that reads x (in the fixed order of the slices: the result is the same on every run)
    int pending_parts = 0;
    bool pending_assign = false;
    bool in_draft = false;  // launches are accounted to the drafter's classes
    bool status_ready = false;   // the status word in the (caller-owned, uninitialised) workspace has been cleared
    // profiling
    bool prof_on = false;
    std::vector<hipEvent_t> events;
    std::vector<ProfRec> recs;
};

namespace {

int fail(tlt_ctx* ctx, hipError_t e) {
    if (ctx) ctx->hip_error = (int)e;
    return TLT_EHIP;
}

struct Scope {  // brackets one launch with events when profiling is on
    tlt_ctx* ctx;
    hipStream_t s;
    bool on;
    Scope(tlt_ctx* c, hipStream_t st, int cls, double flops, double bytes) : ctx(c), s(st), on(c && c->prof_on) {
        if (!on) return;
        size_t need = (ctx->recs.size() + 1) * 2;
        while (ctx->events.size() < need) {
            hipEvent_t ev;
            if (hipEventCreate(&ev) != hipSuccess) {
                on = false;
                return;
            }
            ctx->events.push_back(ev);
        }
        ctx->recs.push_back({cls, flops, bytes});
        (void)hipEventRecord(ctx->events[need - 2], s);
    }
    ~Scope() {
        if (on) (void)hipEventRecord(ctx->events[ctx->recs.size() * 2 - 1], s);
    }
};

#define TLT_RUN(ctx, s, cls, flops, bytes, expr)          \
    do {                                                  \
        hipError_t e__;                                   \
        {                                                 \
            Scope sc__(ctx, s, cls, flops, bytes);        \
            e__ = (expr);                                 \
        }                                                 \
        if (e__ != hipSuccess) return fail(ctx, e__);     \
    } while (0)

size_t esz_of(const tlt_ctx* c) { return c->cfg.dtype == TLT_F32 ? 4 : 2; }

int run_gemm(tlt_ctx* ctx, hipStream_t s, int out_mode, int M, int N, int K, const void* A, const void* W, void* C) {
    const double e = (double)esz_of(ctx);
    const double out_b = out_mode == OUT_T ? e : (out_mode == OUT_F32 ? 4.0 : 8.0);
    TLT_RUN(ctx, s, ctx->in_draft ? CLS_GEMM_DRAFT : CLS_GEMM, 2.0 * M * N * K, ((double)M * K + (double)N * K) * e + (double)M * N * out_b,
            gemm(s, ctx->cfg.dtype, out_mode, M, N, K, A, W, C));
    return TLT_OK;
}

unsigned int* status_word(tlt_ctx* ctx) { return (unsigned int*)(ctx->ws + ctx->plan.status); }

// The status word is cleared by the first call that may raise it (the workspace arrives uninitialised).
int ensure_status(tlt_ctx* ctx, hipStream_t s) {
    if (ctx->status_ready) return TLT_OK;
    hipError_t e = zero_f32(s, 64, (float*)status_word(ctx));
    if (e != hipSuccess) return fail(ctx, e);
    ctx->status_ready = true;
    return TLT_OK;
}

// A W^T as partial products in the workspace (see gemm_parts); returns their number through n_parts.
int run_gemm_parts(tlt_ctx* ctx, hipStream_t s, int M, int N, int K, const void* A, const void* W, int* n_parts) {
    const double e = (double)esz_of(ctx);
    hipError_t err;
    {
        Scope sc(ctx, s, ctx->in_draft ? CLS_GEMM_DRAFT : CLS_GEMM, 2.0 * M * N * K, ((double)M * K + (double)N * K) * e + (double)M * N * 4.0);
        err = gemm_parts(s, ctx->cfg.dtype, M, N, K, A, W, (float*)(ctx->ws + ctx->plan.parts), ctx->plan.parts_bytes, n_parts);
    }
    if (err != hipSuccess) return fail(ctx, err);
    return TLT_OK;
}

// x absorbs the partial products still pending (standalone: where no norm kernel follows that could do it).
int fold_pending(tlt_ctx* ctx, hipStream_t s, int M) {
    if (ctx->pending_parts == 0) return TLT_OK;
    const int h = ctx->cfg.hidden;
    TLT_RUN(ctx, s, CLS_OTHER, 0, (double)M * h * 4 * (2 + ctx->pending_parts),
            add_parts(s, (int64_t)M * h, (float*)(ctx->ws + ctx->plan.x), (const float*)(ctx->ws + ctx->plan.parts), ctx->pending_parts,
                      ctx->pending_assign));
    ctx->pending_parts = 0;
    ctx->pending_assign = false;
    return TLT_OK;
}

// out = rmsnorm(x) * gamma over M rows of the residual stream, x first absorbing what is pending for its x_rows rows (0: M; with
// another io, for the rows that the norm reads: the others are dropped).
int norm_x(tlt_ctx* ctx, hipStream_t s, int M, const void* gamma, void* out, const NormIO& io = NormIO(), int x_rows = 0) {
    const tlt_model_cfg& c = ctx->cfg;
    float* x = (float*)(ctx->ws + ctx->plan.x);
    const double e = (double)esz_of(ctx);
    const int n = ctx->pending_parts;
    const bool assign = ctx->pending_assign;
    ctx->pending_parts = 0;
    ctx->pending_assign = false;
    TLT_RUN(ctx, s, CLS_OTHER, 0, (double)M * c.hidden * ((n > 0 ? 8 : 4) + 4 * n + e),
            rmsnorm(s, c.dtype, M, c.hidden, x, gamma, c.rms_eps, out, io, n > 0 ? ctx->ws + ctx->plan.parts : nullptr, true, n,
                    x_rows > 0 ? x_rows : M, assign));
    return TLT_OK;
}

// The norm of the M rows of the stream for a product that normalises its own rows (gemm_f32_norm_supported): what is pending is absorbed on
// the way, and the rows go to x_out.  Nothing is pending afterwards.
NormIn norm_in(tlt_ctx* ctx, const float* x, const void* gamma, float* x_out) {
    NormIn n;
    n.x = x;
    n.add = ctx->pending_parts > 0 ? (const float*)(ctx->ws + ctx->plan.parts) : nullptr;   // (fp32 mode: one product)
    n.gamma = (const float*)gamma;
    n.eps = ctx->cfg.rms_eps;
    n.assign = ctx->pending_assign;
    n.x_out = x_out;
    return n;
}
void absorbed(tlt_ctx* ctx) {
    ctx->pending_parts = 0;
    ctx->pending_assign = false;
}

// The final norm and the LM head, the stream's rows kept in io's copy rows (or not at all).
int norm_lm_head(tlt_ctx* ctx, hipStream_t s, int M, const NormIO& io, float* logits);

KVLayer kv_layer(const tlt_ctx* ctx, const tlt_kv* kv, int layer) {
    const tlt_model_cfg& c = ctx->cfg;
    KVLayer k;
    const size_t per_layer = (size_t)kv->n_pages * c.n_kv_heads * c.page_size * c.head_dim * esz_of(ctx);
    k.k = (char*)kv->k_pool + per_layer * layer;
    k.v = (char*)kv->v_pool + per_layer * layer;
    k.n_pages = kv->n_pages;
    k.block_table = kv->block_table;
    k.seq_len = kv->seq_len;
    k.max_pages = kv->max_pages;
    k.page_size = c.page_size;
    k.n_kv = c.n_kv_heads;
    k.d = c.head_dim;
    k.seq_len_bound = kv->seq_len_bound;
    return k;
}

// Rows of a block whose output is wanted: row `row` of every `n` (B of them), or none (B = 0).  The block's keys and values are written for all rows.
struct WantedRows {
    int B, n, row;
};

// One decoder block over M = rows.B * rows.n rows whose residual stream sits in the workspace's x.
// later_layer: an earlier layer of the same forward (same rows, same sequence lengths) has left the attention work list
// and the rotary table in the workspace.
// With `wanted` (the last block of a forward only) the stream holds the wanted rows alone, densely, afterwards.
int layer_forward(tlt_ctx* ctx, hipStream_t s, const tlt_layer_weights& w, const Rows& rows, const KVLayer& kv,
                  bool later_layer = false, const WantedRows* wanted = nullptr) {
    const tlt_model_cfg& c = ctx->cfg;
    const Plan& p = ctx->plan;
    char* ws = ctx->ws;
    int M = rows.B * rows.n;
    const int h = c.hidden, F = c.mlp, dt = c.dtype;
    const int q_dim = c.n_q_heads * c.head_dim, qkv_dim = q_dim + 2 * c.n_kv_heads * c.head_dim;
    const double e = (double)esz_of(ctx);
    float* x = (float*)(ws + p.x);
    int rc;
    float* parts = (float*)(ws + p.parts);
    int n_parts = 1;
    RopeTable tab;   // (the drafter is one layer: nothing to keep)
    if (!ctx->in_draft) tab.cs = (float*)(ws + p.rope_cs), tab.at = (int64_t*)(ws + p.rope_at);
    // fp32 mode with few rows: both norms belong to the products behind them.  The stream's rows then go to xn and, at the second norm, back.
    float* x1 = (float*)(ws + p.xn);
    const NormIn n1 = norm_in(ctx, x, w.attn_norm, x1);
    const bool own_norm = !wanted && ctx->pending_parts <= 1 && gemm_f32_norm_supported(dt, M, qkv_dim, h, n1, w.wqkv, nullptr) &&
                          gemm_f32_norm_supported(dt, M, F, h, n1, w.wg, w.wu) && ((uintptr_t)w.mlp_norm & 15) == 0;
    if (own_norm) {
        TLT_RUN(ctx, s, ctx->in_draft ? CLS_GEMM_DRAFT : CLS_GEMM, 2.0 * M * qkv_dim * h, ((double)M * h * 3 + (double)qkv_dim * (h + M)) * e,
                gemm_f32_norm(s, M, qkv_dim, h, n1, w.wqkv, ws + p.qkv));
        absorbed(ctx);
    } else if ((rc = norm_x(ctx, s, M, w.attn_norm, ws + p.xn))) {
        return rc;
    }
    // few rows per sequence in fp32 mode: the attention kernel rotates them and writes them to the cache
    const bool own_rope = !wanted && attention_rope_supported(dt, rows, kv, ws + p.qkv, w.bqkv);
    if (own_norm) {
        if (!own_rope)
            TLT_RUN(ctx, s, CLS_OTHER, 0, (double)M * qkv_dim * e * 2,
                    rope_kv_write(s, dt, rows, kv, ws + p.qkv, c.n_q_heads, c.rope_theta, w.bqkv, tab, later_layer));
    } else if (dt == TLT_BF16 && qkv_dim % 128 == 0 && (size_t)M * qkv_dim * 4 * 2 <= p.parts_bytes &&
        (M <= 256 || gemm_parts_pays(dt, M, qkv_dim, h))) {
        // too few tiles for the chip unless the projection is cut along K, which leaves fp32 partial products;
        // the rotary kernel sums them, rounds the sums to the model dtype, as a product stored once is, and rotates (always up to
        // 256 rows, one row of tiles; above where the cost model of the cuts expects it to pay: a few hundred rows).
        if ((rc = run_gemm_parts(ctx, s, M, qkv_dim, h, ws + p.xn, w.wqkv, &n_parts))) return rc;
        TLT_RUN(ctx, s, CLS_OTHER, 0, (double)M * qkv_dim * (4 * n_parts + e),
                rope_kv_write(s, dt, rows, kv, ws + p.qkv, c.n_q_heads, c.rope_theta, w.bqkv, tab, later_layer, parts, n_parts));
    } else {
        if ((rc = run_gemm(ctx, s, OUT_T, M, qkv_dim, h, ws + p.xn, w.wqkv, ws + p.qkv))) return rc;
        if (!own_rope)
            TLT_RUN(ctx, s, CLS_OTHER, 0, (double)M * qkv_dim * e * 2,
                    rope_kv_write(s, dt, rows, kv, ws + p.qkv, c.n_q_heads, c.rope_theta, w.bqkv, tab, later_layer));
    }
    if (wanted && wanted->B == 0) {
        ctx->pending_parts = 0;
        return TLT_OK;
    }
    const char* att = ws + p.att;
    {
        // algorithmic traffic: one pass over the cached K and V of every sequence (bounded by the
        // host-known length) plus q in / out; flops: 4 * d per (query row, head, key)
        const double keys = (double)rows.B * ((double)kv.seq_len_bound + rows.n_region);
        const double bytes = keys * 2.0 * c.n_kv_heads * c.head_dim * e + 2.0 * M * q_dim * e;
        const double flops = 4.0 * c.head_dim * c.n_q_heads * (double)rows.n * keys;
        TLT_RUN(ctx, s, ctx->in_draft ? CLS_ATTN_DRAFT : CLS_ATTN, flops, bytes,
                own_rope ? attention_rope(s, rows, kv, ws + p.qkv, ws + p.att, c.n_q_heads, c.rope_theta, w.bqkv, tab, later_layer)
                         : attention(s, dt, rows, kv, ws + p.qkv, ws + p.att, c.n_q_heads, ws + p.attn_ws, p.attn_ws_bytes, ctx->attn_impl,
                                     later_layer, ctx->status_ready ? status_word(ctx) : nullptr));
    }
    if (wanted) {
        // the wanted rows of the stream to its front (by way of xn: source and destination rows may meet), those of the attention to where
        // qkv was; both buffers are sized for all rows
        M = wanted->B;
        const int n = wanted->n, up = n - 1 - wanted->row, att_words = (int)(q_dim * esz_of(ctx) / 4);
        TLT_RUN(ctx, s, CLS_OTHER, 0, (double)M * h * 8, gather_last_rows(s, M, n, h, x - (int64_t)up * h, (float*)(ws + p.xn), 1));
        TLT_RUN(ctx, s, CLS_OTHER, 0, (double)M * h * 8, copy_f32(s, (int64_t)M * h, (const float*)(ws + p.xn), x));
        TLT_RUN(ctx, s, CLS_OTHER, 0, (double)M * q_dim * e * 2,
                gather_last_rows(s, M, n, att_words, (const float*)att - (int64_t)up * att_words, (float*)(ws + p.qkv), 1));
        att = ws + p.qkv;
    }
    // the output projection's product (fp32, possibly several partial products of a K split) joins the
    // residual stream inside the norm kernel that follows: plain stores in the GEMM's epilogue instead of
    // a read-modify-write of the stream by every tile, and a sum formed in a fixed order
    if (dt == TLT_BF16 && !ctx->oproj_f32 && M > 256) {   // (measurement switch: the product rounded to the model dtype)
        if ((rc = run_gemm(ctx, s, OUT_T, M, h, q_dim, att, w.wo, parts))) return rc;
        TLT_RUN(ctx, s, CLS_OTHER, 0, (double)M * h * (8 + 2 * e),
                rmsnorm(s, dt, M, h, x, w.mlp_norm, c.rms_eps, ws + p.xn, NormIO(), parts, false, 1, M));
    } else {
        if ((rc = run_gemm_parts(ctx, s, M, h, q_dim, att, w.wo, &n_parts))) return rc;
        ctx->pending_parts = n_parts;
        ctx->pending_assign = false;
        if (!own_norm && (rc = norm_x(ctx, s, M, w.mlp_norm, ws + p.xn))) return rc;
    }
    if (own_norm) {
        TLT_RUN(ctx, s, ctx->in_draft ? CLS_GEMM_DRAFT : CLS_GEMM, 4.0 * M * F * h, ((double)M * h * 3 + 2.0 * F * h + (double)M * F) * e,
                gemm_f32_norm_glu(s, M, F, h, norm_in(ctx, x1, w.mlp_norm, x), w.wg, w.wu, ws + p.act));
        absorbed(ctx);
    } else if (gemm_glu_supported(dt, M, F, h, ws + p.xn, w.wg, w.wu)) {
        TLT_RUN(ctx, s, ctx->in_draft ? CLS_GEMM_DRAFT : CLS_GEMM, 4.0 * M * F * h,
                ((double)M * h + 2.0 * F * h + (double)M * F) * e, gemm_glu(s, dt, M, F, h, ws + p.xn, w.wg, w.wu, ws + p.act));
    } else {
        if ((rc = run_gemm(ctx, s, OUT_T, M, F, h, ws + p.xn, w.wg, ws + p.g))) return rc;
        if ((rc = run_gemm(ctx, s, OUT_T, M, F, h, ws + p.xn, w.wu, ws + p.u))) return rc;
        TLT_RUN(ctx, s, CLS_OTHER, 0, (double)M * F * e * 3, swiglu(s, dt, (int64_t)M * F, ws + p.g, ws + p.u, ws + p.act));
    }
    // the down projection's product stays pending: the next kernel that reads the stream absorbs it
    if ((rc = run_gemm_parts(ctx, s, M, h, F, ws + p.act, w.wd, &n_parts))) return rc;
    ctx->pending_parts = n_parts;
    ctx->pending_assign = false;
    return TLT_OK;
}

int norm_lm_head(tlt_ctx* ctx, hipStream_t s, int M, const NormIO& io, float* logits) {
    const tlt_model_cfg& c = ctx->cfg;
    NormIn n = norm_in(ctx, (const float*)(ctx->ws + ctx->plan.x), ctx->target.final_norm, io.copy);
    n.out_n = io.copy_n;
    n.out_stride = io.copy_stride;
    n.out_base = io.copy_base;
    if (ctx->pending_parts <= 1 && gemm_f32_norm_supported(c.dtype, M, c.vocab, c.hidden, n, ctx->target.lm_head, nullptr)) {
        TLT_RUN(ctx, s, ctx->in_draft ? CLS_GEMM_DRAFT : CLS_GEMM, 2.0 * M * c.vocab * c.hidden,
                ((double)M * c.hidden * 3 + (double)c.vocab * (c.hidden + M)) * 4, gemm_f32_norm(s, M, c.vocab, c.hidden, n, ctx->target.lm_head, logits));
        absorbed(ctx);
        return TLT_OK;
    }
    int rc = norm_x(ctx, s, M, ctx->target.final_norm, ctx->ws + ctx->plan.xn, io);
    return rc ? rc : run_gemm(ctx, s, OUT_F32, M, c.vocab, c.hidden, ctx->ws + ctx->plan.xn, ctx->target.lm_head, logits);
}

int check_kv(const tlt_ctx* ctx, const tlt_kv* kv, int new_rows) {
    if (!kv || !kv->k_pool || !kv->v_pool || !kv->block_table || !kv->seq_len || kv->n_pages < 1 || kv->max_pages < 1 ||
        kv->seq_len_bound < 0)
        return TLT_EINVAL;
    if ((int64_t)kv->seq_len_bound + new_rows > (int64_t)kv->max_pages * ctx->cfg.page_size) return TLT_ENOPAGES;
    if (kv->seq_len_bound + new_rows > ctx->max_ctx) return TLT_ESHAPE;
    return TLT_OK;
}

bool tree_ok(const tlt_tree* t) { return t && t->token && t->parent && t->depth && t->anc_mask && t->n >= 1 && t->n <= TLT_MAX_TREE; }

}  // namespace

extern "C" {

const char* tlt_strerror(int code) {
    switch (code) {
        case TLT_OK: return "ok";
        case TLT_EINVAL: return "invalid argument";
        case TLT_ESHAPE: return "size exceeds the limits given to tlt_create (or workspace too small)";
        case TLT_ENOPAGES: return "block table too short for seq_len_bound + new rows";
        case TLT_EHIP: return "HIP call failed";
        case TLT_ENOTIMPL: return "not implemented";
        case TLT_ESYNC: return "workgroups of a kernel could not meet on the device (chip busy with other work)";
        default: return "unknown error";
    }
}

int tlt_last_hip_error(const tlt_ctx* ctx) { return ctx ? ctx->hip_error : 0; }

size_t tlt_workspace_bytes(const tlt_model_cfg* cfg, int max_batch, int max_n, int max_depth, int max_topk, int max_ctx) {
    Plan p;
    if (!cfg_ok(cfg) || !plan_workspace(*cfg, max_batch, max_n, max_depth, max_topk, max_ctx, p)) return 0;
    return p.total;
}

int tlt_create(tlt_ctx** out, const tlt_model_cfg* cfg, const tlt_weights* target, const tlt_weights* draft, int max_batch,
               int max_n, int max_depth, int max_topk, int max_ctx, void* workspace, size_t workspace_bytes) {
    if (!out || !cfg_ok(cfg) || !target || !target->embed || !target->lm_head || !target->final_norm || !target->layers ||
        !workspace)
        return TLT_EINVAL;
    if (((uintptr_t)workspace & 255) != 0) return TLT_EINVAL;
    Plan p;
    if (!plan_workspace(*cfg, max_batch, max_n, max_depth, max_topk, max_ctx, p)) return TLT_EINVAL;
    if (workspace_bytes < p.total) return TLT_ESHAPE;
    for (int l = 0; l < cfg->n_layers; ++l) {
        const tlt_layer_weights& w = target->layers[l];
        if (!w.attn_norm || !w.wqkv || !w.wo || !w.mlp_norm || !w.wg || !w.wu || !w.wd) return TLT_EINVAL;
    }
    if (draft) {
        if (!draft->fc || !draft->layers) return TLT_EINVAL;
        const tlt_layer_weights& w = draft->layers[0];
        if (!w.attn_norm || !w.wqkv || !w.wo || !w.mlp_norm || !w.wg || !w.wu || !w.wd) return TLT_EINVAL;
    }
    tlt_ctx* c = new (std::nothrow) tlt_ctx();
    if (!c) return TLT_EINVAL;
    c->cfg = *cfg;
    c->target = *target;
    c->target_layers.assign(target->layers, target->layers + cfg->n_layers);
    c->target.layers = c->target_layers.data();
    if (draft) {
        c->have_draft = true;
        c->draft = *draft;
        c->draft_layers.assign(draft->layers, draft->layers + 1);
        c->draft.layers = c->draft_layers.data();
    }
    c->max_batch = max_batch;
    c->max_n = max_n;
    c->max_depth = max_depth;
    c->max_topk = max_topk;
    c->max_ctx = max_ctx;
    c->ws = (char*)workspace;
    c->plan = p;
    *out = c;
    return TLT_OK;
}

int tlt_destroy(tlt_ctx* ctx) {
    if (!ctx) return TLT_EINVAL;
    for (hipEvent_t e : ctx->events) (void)hipEventDestroy(e);
    delete ctx;
    return TLT_OK;
}

int tlt_set_attention_impl(tlt_ctx* ctx, int impl) {
    if (!ctx) return TLT_EINVAL;
    ctx->attn_impl = impl;
    return TLT_OK;
}

int tlt_device_status(tlt_ctx* ctx, void* stream, uint32_t* flags) {
    if (!ctx) return TLT_EINVAL;
    if (flags) *flags = 0;
    if (!ctx->status_ready) return TLT_OK;   // nothing that could raise it has run
    hipStream_t s = (hipStream_t)stream;
    uint32_t host = 0;
    hipError_t e = hipMemcpyAsync(&host, status_word(ctx), sizeof(host), hipMemcpyDeviceToHost, s);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return fail(ctx, e);
    if (flags) *flags = host;
    if (host != 0) {
        e = zero_f32(s, 64, (float*)status_word(ctx));
        if (e != hipSuccess) return fail(ctx, e);
    }
    return (host & TLT_STATUS_CONTEXT_TRUNCATED) ? TLT_ESHAPE : ((host & TLT_STATUS_NO_RENDEZVOUS) ? TLT_ESYNC : TLT_OK);
}

// The address at which kernels reach a word of the caller's pinned (or managed) host memory; null for any other memory (a kernel
// that stored there would fault).  Asked of the runtime at every call: what an address belongs to may change between two.
static int32_t* mapped_host_word(int32_t* p) {
    hipPointerAttribute_t a = {};
    if (hipPointerGetAttributes(&a, p) != hipSuccess) {
        (void)hipGetLastError();   // (memory that the runtime does not know: not an error of the next call)
        return nullptr;
    }
    return a.type == hipMemoryTypeHost || a.type == hipMemoryTypeManaged ? (int32_t*)a.devicePointer : nullptr;
}

int tlt_step_report(tlt_ctx* ctx, void* stream, const int32_t* words, int n, int32_t* out, uint32_t* flags) {
    if (!ctx || !words || n < 1 || n > (1 << 24) || !out) return TLT_EINVAL;
    int32_t* const dst = mapped_host_word(out);
    if (!dst || mapped_host_word(out + n) != dst + n) return TLT_EINVAL;
    if (flags) *flags = 0;
    hipStream_t s = (hipStream_t)stream;
    hipError_t e = report_words(s, n, words, ctx->status_ready ? status_word(ctx) : nullptr, dst);
    if (e == hipSuccess) e = hipStreamSynchronize(s);
    if (e != hipSuccess) return fail(ctx, e);
    const uint32_t raised = (uint32_t)out[n];
    if (flags) *flags = raised;
    if (raised != 0 && (e = zero_f32(s, 64, (float*)status_word(ctx))) != hipSuccess) return fail(ctx, e);
    return (raised & TLT_STATUS_CONTEXT_TRUNCATED) ? TLT_ESHAPE : ((raised & TLT_STATUS_NO_RENDEZVOUS) ? TLT_ESYNC : TLT_OK);
}

int tlt_set_oproj_rounding(tlt_ctx* ctx, int round_to_model_dtype) {
    if (!ctx) return TLT_EINVAL;
    ctx->oproj_f32 = round_to_model_dtype == 0;
    return TLT_OK;
}

int tlt_tree_finalize(tlt_ctx* ctx, void* stream, int B, tlt_tree* tree) {
    if (!ctx || !tree_ok(tree) || B < 1) return TLT_EINVAL;
    hipStream_t s = (hipStream_t)stream;
    TLT_RUN(ctx, s, CLS_OTHER, 0, 0, tree_finalize(s, B, tree->n, tree->parent, tree->depth, tree->anc_mask));
    return TLT_OK;
}

int tlt_verify_forward(tlt_ctx* ctx, void* stream, int B, const tlt_tree* tree, tlt_kv* kv, float* out_logits,
                       int32_t* out_argmax, float* out_lse, float* out_hidden) {
    if (!ctx || !tree_ok(tree) || B < 1) return TLT_EINVAL;
    if (B > ctx->max_batch || tree->n > ctx->max_n) return TLT_ESHAPE;
    int rc = check_kv(ctx, kv, tree->n);
    if (rc) return rc;
    hipStream_t s = (hipStream_t)stream;
    if ((rc = ensure_status(ctx, s))) return rc;
    ctx->pending_parts = 0;   // (nothing of an earlier call is pending: every call absorbs what it leaves)
    const tlt_model_cfg& c = ctx->cfg;
    const Plan& p = ctx->plan;
    char* ws = ctx->ws;
    const int n = tree->n, M = B * n, h = c.hidden, V = c.vocab;
    const double e = (double)esz_of(ctx);
    float* x = (float*)(ws + p.x);

    TLT_RUN(ctx, s, CLS_OTHER, 0, (double)M * h * (e + 4), embed_rows(s, c.dtype, M, h, V, tree->token, ctx->target.embed, x));
    Rows rows;
    rows.B = B;
    rows.n = n;
    rows.pos_off = tree->depth;
    rows.mask = tree->anc_mask;
    rows.mask_words = 1;
    rows.n_region = n;
    for (int l = 0; l < c.n_layers; ++l) {
        rc = layer_forward(ctx, s, ctx->target.layers[l], rows, kv_layer(ctx, kv, l), l > 0);
        if (rc) return rc;
    }
    // (the last block's down projection is still pending: the final norm absorbs it into x, or, when no logits
    // are wanted, a plain add)
    if (out_logits || out_argmax || out_lse) {
        float* logits = out_logits ? out_logits : (float*)(ws + p.logits);
        NormIO io;
        io.copy = out_hidden;   // (the stream ends here: its rows leave x for the caller's buffer on the way, where that is wanted)
        if (!out_logits && !out_lse && gemm_argmax_supported(c.dtype, M, V, h, ws + p.xn, ctx->target.lm_head)) {
            if ((rc = norm_x(ctx, s, M, ctx->target.final_norm, ws + p.xn, io))) return rc;
            // only the most likely tokens are wanted: the logits never leave the LM head's registers
            // (block partials go where the logits would have gone: M * V/128 * 8 bytes of M * V * 4)
            TLT_RUN(ctx, s, CLS_GEMM, 2.0 * M * V * h, ((double)M * h + (double)V * h) * e,
                    gemm_argmax(s, M, V, h, ws + p.xn, ctx->target.lm_head, logits, out_argmax));
        } else {
            if ((rc = norm_lm_head(ctx, s, M, io, logits))) return rc;
            if (out_argmax) TLT_RUN(ctx, s, CLS_OTHER, 0, (double)M * V * 4, row_argmax(s, M, V, logits, out_argmax, ws + p.parts, p.parts_bytes));   // (nothing is pending: the slices' buffer is idle)
            if (out_lse) TLT_RUN(ctx, s, CLS_OTHER, 0, (double)M * V * 8, row_lse(s, M, V, logits, out_lse));
        }
    } else {
        if ((rc = fold_pending(ctx, s, M))) return rc;
        if (out_hidden) TLT_RUN(ctx, s, CLS_OTHER, 0, (double)M * h * 8, copy_f32(s, (int64_t)M * h, x, out_hidden));
    }
    return TLT_OK;
}

// x = fc([embedding ; hidden]) of the drafter (2h -> h), left pending as partial products: with few rows the
// product has far fewer tiles than the chip has CUs while K = 2h is long, so it is cut along K; the
// drafter block's first norm kernel forms x from the slices.
static int draft_fc(tlt_ctx* ctx, hipStream_t s, int M, const void* xin) {
    int n_parts = 1;
    int rc = run_gemm_parts(ctx, s, M, ctx->cfg.hidden, 2 * ctx->cfg.hidden, xin, ctx->draft.fc, &n_parts);
    if (rc) return rc;
    ctx->pending_parts = n_parts;
    ctx->pending_assign = true;
    return TLT_OK;
}

// Drafter catch-up shared by both expansion modes: entries for the newly committed positions, the
// last one's output as feature row 0 and, normalised, in the workspace's xn, committed length advanced.
static int draft_extend_rows(tlt_ctx* ctx, hipStream_t s, int B, const int32_t* new_tokens, const int32_t* new_src,
                             const int32_t* n_new, int new_stride, const float* hidden, int hidden_n, tlt_kv* draft_kv,
                             KVLayer& kvl) {
    const tlt_model_cfg& c = ctx->cfg;
    const Plan& p = ctx->plan;
    char* ws = ctx->ws;
    const int h = c.hidden, V = c.vocab, dt = c.dtype;
    const double e = (double)esz_of(ctx);
    float* feat = (float*)(ws + p.feat);
    const int FR = p.feat_rows;
    int rc;
    const int M = B * new_stride;
    TLT_RUN(ctx, s, CLS_OTHER, 0, (double)M * h * (4 + 3 * e),
            draft_input(s, dt, B, new_stride, h, V, new_tokens, new_src, n_new, hidden_n, (int64_t)B * hidden_n, hidden,
                        ctx->target.embed, ws + p.xn));
    if ((rc = draft_fc(ctx, s, M, ws + p.xn))) return rc;
    Rows rows;
    rows.B = B;
    rows.n = new_stride;
    rows.n_valid = n_new;
    rows.pos_stride = 1;
    rows.n_region = new_stride;
    if ((rc = layer_forward(ctx, s, ctx->draft.layers[0], rows, kvl))) return rc;
    NormIO io;
    io.n_valid = n_new;
    io.n = new_stride;
    io.copy = feat;
    io.copy_stride = FR;
    io.len = draft_kv->seq_len;
    if ((rc = norm_x(ctx, s, B, ctx->target.final_norm, ws + p.xn, io, M))) return rc;
    kvl.seq_len_bound += new_stride;
    return TLT_OK;
}

// Workspace of a prefill pass of B * C virtual sequences of m rows, carved from what lies in front of the feature rows of the
// ordinary plan: a pass wants no logits, whose room is most of the workspace.
struct PrefillPlan {
    Plan plan;
    size_t tok, nxt, src, n_valid, len_t, len_d, vtab_t, vtab_d;
};
static bool plan_prefill(const tlt_ctx* ctx, int BC, int m, const tlt_kv* kv, const tlt_kv* dkv, int bound, PrefillPlan& q) {
    const tlt_model_cfg& c = ctx->cfg;
    const size_t esz = esz_of(ctx), R = (size_t)BC * m, h = c.hidden, F = c.mlp;
    const size_t q_dim = (size_t)c.n_q_heads * c.head_dim, qkv_dim = q_dim + 2 * (size_t)c.n_kv_heads * c.head_dim;
    Plan& p = q.plan;
    p = ctx->plan;   // (feature rows and status word stay where they are)
    size_t o = 0;
    auto take = [&](size_t bytes) {
        const size_t at = o;
        o = align_up(o + bytes);
        return at;
    };
    p.max_rows = (int)R;
    p.x = take(R * h * 4);
    p.xn = take(R * 2 * h * esz);
    p.qkv = take(R * qkv_dim * esz);
    p.rope_cs = take(R * (size_t)c.head_dim * 4);
    p.rope_at = take(R * 8);
    p.att = take(R * q_dim * esz);
    p.act = take(R * F * esz);
    bool fused = true;   // (else gate and up need buffers of their own)
    auto takes = [&](const tlt_layer_weights& w) { return gemm_glu_supported(c.dtype, (int)R, c.mlp, c.hidden, ctx->ws, w.wg, w.wu); };
    for (int l = 0; l < c.n_layers; ++l) fused = fused && takes(ctx->target.layers[l]);
    fused = fused && takes(ctx->draft.layers[0]);
    p.g = take(fused ? 0 : R * F * esz);
    p.u = take(fused ? 0 : R * F * esz);
    q.tok = take(R * 4);
    q.nxt = take(R * 4);
    q.src = take(R * 4);
    q.n_valid = take((size_t)BC * 4);
    q.len_t = take((size_t)BC * 4);
    q.len_d = take((size_t)BC * 4);
    q.vtab_t = take((size_t)BC * kv->max_pages * 4);
    q.vtab_d = take((size_t)BC * dkv->max_pages * 4);
    p.attn_ws_bytes = attention_workspace_bytes(BC, m, c.n_q_heads, c.n_kv_heads, c.head_dim, bound);
    p.attn_ws = take(p.attn_ws_bytes);
    // partial products: what is left, up to what any plan of cuts asks for; three slices of the widest at the least
    const size_t slice = R * std::max(h, qkv_dim) * 4, want = (c.dtype == TLT_BF16 ? 3 : 1) * slice;
    p.parts = o;
    if (o + want > ctx->plan.feat) return false;
    p.parts_bytes = std::min(ctx->plan.feat - o, std::max(want, 12 * slice));
    return true;
}

// Rows of a pass: what a product of this model's widths needs to run at the rate of large ones (7B shape, 4 prompts of 301 tokens:
// five passes of 256 rows 27.5 ms, one of 1200 15.9).  Four blocks of that shape, ms with at most 1024 / 2048 / 4096 rows: 4 x 301 3.17 /
// 2.56 / 2.57, 8 x 250 4.31 / 3.94 / 3.94, 8 x 600 10.6 / 9.6 / 9.8, 16 x 257 10.4 (no two chunks fit) / 7.7 / 8.5; a single prompt of 2049 to
// 4097 the same (its engine's workspace holds fewer rows).
constexpr int kPrefillRows = 2048;

int tlt_prefill(tlt_ctx* ctx, void* stream, int B, int n_tokens, int chunk, const int32_t* tokens, int token_stride, tlt_kv* kv,
                tlt_kv* draft_kv) {
    if (!ctx || !ctx->have_draft || B < 1 || n_tokens < 1 || chunk < 1 || !tokens || token_stride <= n_tokens) return TLT_EINVAL;
    if (B > ctx->max_batch || chunk > ctx->max_n) return TLT_ESHAPE;
    int rc;
    if ((rc = check_kv(ctx, kv, n_tokens)) || (rc = check_kv(ctx, draft_kv, n_tokens))) return rc;
    // chunks of equal length, and as many of each sequence in a pass as the workspace holds
    int nc = (n_tokens + chunk - 1) / chunk;
    const int m = (n_tokens + nc - 1) / nc;
    nc = (n_tokens + m - 1) / m;
    const int bound = std::max(kv->seq_len_bound, draft_kv->seq_len_bound) + n_tokens;
    PrefillPlan q;
    int C = std::min(nc, std::max(1, kPrefillRows / (B * m)));
    while (C > 1 && !plan_prefill(ctx, B * C, m, kv, draft_kv, bound, q)) --C;
    if (C < 2) return TLT_ENOTIMPL;
    C = (nc + (nc + C - 1) / C - 1) / ((nc + C - 1) / C);   // (as many passes, evenly filled)
    if (!plan_prefill(ctx, B * C, m, kv, draft_kv, bound, q)) return TLT_ENOTIMPL;

    hipStream_t s = (hipStream_t)stream;
    if ((rc = ensure_status(ctx, s))) return rc;
    struct PlanSwap {   // the block's kernels find the pass's buffers where they find a step's
        tlt_ctx* c;
        Plan saved;
        PlanSwap(tlt_ctx* x, const Plan& p) : c(x), saved(x->plan) { c->plan = p; }
        ~PlanSwap() {
            c->plan = saved;
            c->in_draft = false;
        }
    } swap(ctx, q.plan);
    const tlt_model_cfg& c = ctx->cfg;
    const Plan& p = ctx->plan;
    char* ws = ctx->ws;
    const int h = c.hidden, V = c.vocab;
    const double e = (double)esz_of(ctx);
    float* x = (float*)(ws + p.x);
    PrefillPass pass;
    pass.tokens = tokens;
    pass.token_stride = token_stride;
    pass.n_tokens = n_tokens;
    pass.m = m;
    pass.seq_len_t = kv->seq_len;
    pass.seq_len_d = draft_kv->seq_len;
    pass.table_t = kv->block_table;
    pass.table_d = draft_kv->block_table;
    pass.pages_t = kv->max_pages;
    pass.pages_d = draft_kv->max_pages;
    pass.tok = (int32_t*)(ws + q.tok);
    pass.nxt = (int32_t*)(ws + q.nxt);
    pass.src = (int32_t*)(ws + q.src);
    pass.n_valid = (int32_t*)(ws + q.n_valid);
    pass.len_t = (int32_t*)(ws + q.len_t);
    pass.len_d = (int32_t*)(ws + q.len_d);
    pass.vtab_t = (int32_t*)(ws + q.vtab_t);
    pass.vtab_d = (int32_t*)(ws + q.vtab_d);
    auto virtual_kv = [&](const tlt_kv* of, int32_t* lens, int32_t* table) {
        tlt_kv v = *of;
        v.seq_len = lens;
        v.block_table = table;
        v.seq_len_bound = of->seq_len_bound + n_tokens - 1;
        return v;
    };
    const tlt_kv vt = virtual_kv(kv, pass.len_t, pass.vtab_t), vd = virtual_kv(draft_kv, pass.len_d, pass.vtab_d);
    for (int done = 0; done < n_tokens;) {
        const int left = (n_tokens - done + m - 1) / m, Cp = std::min(C, left), BC = B * Cp, M = BC * m;
        const int taken = std::min(Cp * m, n_tokens - done);
        pass.done = done;
        pass.C = Cp;
        ctx->pending_parts = 0;
        TLT_RUN(ctx, s, CLS_OTHER, 0, 0, prefill_rows(s, B, pass));
        TLT_RUN(ctx, s, CLS_OTHER, 0, (double)M * h * (e + 4), embed_rows(s, c.dtype, M, h, V, pass.tok, ctx->target.embed, x));
        Rows rows;   // causal within a chunk
        rows.B = BC;
        rows.n = m;
        rows.n_valid = pass.n_valid;
        rows.pos_stride = 1;
        rows.n_region = m;
        rows.shared_ctx = Cp > 1;
        for (int l = 0; l < c.n_layers; ++l)
            if ((rc = layer_forward(ctx, s, ctx->target.layers[l], rows, kv_layer(ctx, &vt, l), l > 0))) return rc;
        if ((rc = fold_pending(ctx, s, M))) return rc;
        // the drafter's entries of the same positions, from the hidden states in x
        ctx->in_draft = true;
        TLT_RUN(ctx, s, CLS_OTHER, 0, (double)M * h * (4 + 3 * e),
                draft_input(s, c.dtype, BC, m, h, V, pass.nxt, pass.src, pass.n_valid, m, (int64_t)M, x, ctx->target.embed, ws + p.xn));
        if ((rc = draft_fc(ctx, s, M, ws + p.xn))) return rc;
        // only the prompt's last position's output is wanted, as feature row 0 (4 prompts x 301 tokens: the block's other 1196 rows cost
        // 0.4 ms of 16.2 behind its keys and values)
        const bool last = done + taken == n_tokens;
        const WantedRows wanted{last ? B : 0, Cp * m, taken - 1};
        if ((rc = layer_forward(ctx, s, ctx->draft.layers[0], rows, kv_layer(ctx, &vd, 0), false, &wanted))) return rc;
        ctx->in_draft = false;
        done += taken;
        if (last) {
            if ((rc = fold_pending(ctx, s, B))) return rc;
            TLT_RUN(ctx, s, CLS_OTHER, 0, (double)B * h * 8, gather_last_rows(s, B, 1, h, x, (float*)(ws + p.feat), p.feat_rows));
        }
        ctx->pending_parts = 0;
        TLT_RUN(ctx, s, CLS_OTHER, 0, 0, add_i32(s, B, kv->seq_len, nullptr, taken));
        TLT_RUN(ctx, s, CLS_OTHER, 0, 0, add_i32(s, B, draft_kv->seq_len, nullptr, taken));
    }
    return TLT_OK;
}

int tlt_draft_expand(tlt_ctx* ctx, void* stream, int B, int depth, int topk, int n_verify, int mode,
                     const int32_t* new_tokens, const int32_t* new_src, const int32_t* n_new, int new_stride,
                     const float* hidden, int hidden_n, const int32_t* root_tokens, tlt_kv* draft_kv, tlt_tree* out_tree) {
    if (!ctx || !ctx->have_draft || B < 1 || depth < 0 || new_stride < 0) return TLT_EINVAL;
    if (mode != 0) return TLT_ENOTIMPL;
    const bool do_extend = new_stride > 0;
    const bool do_expand = depth >= 1 && out_tree != nullptr;
    if (do_extend && (!new_tokens || !new_src || !n_new || !hidden || hidden_n < 1)) return TLT_EINVAL;
    if (do_expand && (!tree_ok(out_tree) || !out_tree->score || (!root_tokens && !do_extend) || topk < 1 || n_verify < 1))
        return TLT_EINVAL;
    if (B > ctx->max_batch || new_stride > std::max(ctx->max_n, ctx->max_topk)) return TLT_ESHAPE;
    if (do_expand && (depth > ctx->max_depth || topk > ctx->max_topk || n_verify > ctx->max_n)) return TLT_ESHAPE;
    // a provisional drafter row is one bit of a 128-bit visibility mask
    if (do_expand && (depth - 1) * topk > kMaxProvisionalRows) return TLT_ESHAPE;
    const int pool_n = do_expand ? topk + (depth - 1) * topk * topk : 0;
    if (do_expand && out_tree->n != std::min(n_verify, 1 + pool_n)) return TLT_EINVAL;
    const int prov_rows = do_expand ? (depth - 1) * topk : 0;
    int rc = check_kv(ctx, draft_kv, new_stride + prov_rows);
    if (rc) return rc;

    struct DraftFlag {
        tlt_ctx* c;
        explicit DraftFlag(tlt_ctx* x) : c(x) { c->in_draft = true; }
        ~DraftFlag() { c->in_draft = false; }
    } draft_flag(ctx);
    hipStream_t s = (hipStream_t)stream;
    if ((rc = ensure_status(ctx, s))) return rc;
    ctx->pending_parts = 0;
    const tlt_model_cfg& c = ctx->cfg;
    const Plan& p = ctx->plan;
    char* ws = ctx->ws;
    const int h = c.hidden, V = c.vocab, dt = c.dtype;
    const double e = (double)esz_of(ctx);
    float* feat = (float*)(ws + p.feat);
    float* logits = (float*)(ws + p.logits);
    const int FR = p.feat_rows;
    const tlt_layer_weights& lw = ctx->draft.layers[0];
    KVLayer kvl = kv_layer(ctx, draft_kv, 0);

    if (do_extend && (rc = draft_extend_rows(ctx, s, B, new_tokens, new_src, n_new, new_stride, hidden, hidden_n, draft_kv, kvl)))
        return rc;
    if (!do_expand) return TLT_OK;

    DraftState st;
    st.P = p.pool_cap;
    st.pool_token = (int32_t*)(ws + p.pool_token);
    st.pool_score = (float*)(ws + p.pool_score);
    st.pool_parent = (int32_t*)(ws + p.pool_parent);
    st.pool_depth = (int32_t*)(ws + p.pool_depth);
    st.pool_mask = (uint64_t*)(ws + p.pool_mask);
    st.fr_token = (int32_t*)(ws + p.fr_token);
    st.fr_src = (int32_t*)(ws + p.fr_src);
    st.fr_pool = (int32_t*)(ws + p.fr_pool);
    st.fr_mask = (uint64_t*)(ws + p.fr_mask);

    // root distribution: feature row 0 of every sequence -> final norm -> LM head -> top-k
    if (!do_extend) {   // (an extend has left it in xn)
        NormIO io;
        io.src_stride = FR;
        TLT_RUN(ctx, s, CLS_OTHER, 0, (double)B * h * (4 + e), rmsnorm(s, dt, B, h, feat, ctx->target.final_norm, c.rms_eps, ws + p.xn, io));
    }
    if ((rc = run_gemm(ctx, s, OUT_F32, B, V, h, ws + p.xn, ctx->target.lm_head, logits))) return rc;
    TLT_RUN(ctx, s, CLS_OTHER, 0, (double)B * V * 4, draft_level(s, B, topk, 0, V, logits, ws + p.topk_ws, st));

    for (int level = 1; level < depth; ++level) {
        const int M = B * topk;
        TLT_RUN(ctx, s, CLS_OTHER, 0, (double)M * h * (4 + 3 * e),
                draft_input(s, dt, B, topk, h, V, st.fr_token, st.fr_src, nullptr, FR, (int64_t)B * FR, feat,
                            ctx->target.embed, ws + p.xn));
        if ((rc = draft_fc(ctx, s, M, ws + p.xn))) return rc;
        Rows rows;
        rows.B = B;
        rows.n = topk;
        rows.pos_base = level - 1;
        rows.pos_stride = 0;
        rows.slot_base = (level - 1) * topk;
        rows.mask = st.fr_mask;
        rows.mask_words = 2;
        rows.n_region = level * topk;
        if ((rc = layer_forward(ctx, s, lw, rows, kvl))) return rc;
        NormIO io;   // the block's output (x and the pending down projection) goes to the level's feature rows
        io.copy = feat;
        io.copy_n = topk;
        io.copy_stride = FR;
        io.copy_base = 1 + (level - 1) * topk;
        if ((rc = norm_lm_head(ctx, s, M, io, logits))) return rc;
        TLT_RUN(ctx, s, CLS_OTHER, 0, (double)M * V * 4, draft_level(s, B, topk, level, V, logits, ws + p.topk_ws, st));
    }
    TLT_RUN(ctx, s, CLS_OTHER, 0, 0,
            draft_prune(s, B, pool_n, out_tree->n, root_tokens, new_tokens, n_new, new_stride, st, out_tree->token, out_tree->parent, out_tree->depth,
                        out_tree->anc_mask, out_tree->score));
    return TLT_OK;
}

int tlt_draft_pool(tlt_ctx* ctx, void* stream, int B, int depth, int topk, int32_t* token, int32_t* parent, float* score) {
    if (!ctx || !ctx->have_draft || B < 1 || depth < 1 || topk < 1 || !token || !parent || !score) return TLT_EINVAL;
    if (B > ctx->max_batch || depth > ctx->max_depth || topk > ctx->max_topk) return TLT_ESHAPE;
    hipStream_t s = (hipStream_t)stream;
    const Plan& p = ctx->plan;
    const size_t n = (size_t)topk + (size_t)(depth - 1) * topk * topk, src_pitch = (size_t)p.pool_cap * 4;
    const struct {
        void* dst;
        size_t off;
    } parts[3] = {{token, p.pool_token}, {parent, p.pool_parent}, {score, p.pool_score}};
    for (const auto& part : parts) {
        hipError_t e = hipMemcpy2DAsync(part.dst, n * 4, ctx->ws + part.off, src_pitch, n * 4, (size_t)B,
                                        hipMemcpyDeviceToDevice, s);
        if (e != hipSuccess) return fail(ctx, e);
    }
    return TLT_OK;
}

int tlt_draft_sample(tlt_ctx* ctx, void* stream, int B, int depth, int topk, int n_verify, float temperature,
                     const int32_t* new_tokens, const int32_t* new_src, const int32_t* n_new, int new_stride,
                     const float* hidden, int hidden_n, const int32_t* root_tokens, tlt_kv* draft_kv, const uint32_t* u_draw,
                     tlt_tree* out_tree, float* out_draft_q) {
    if (!ctx || !ctx->have_draft || B < 1 || depth < 1 || new_stride < 0 || topk < 1 || n_verify < 1 || !(temperature > 0.f))
        return TLT_EINVAL;
    const bool do_extend = new_stride > 0;
    if (do_extend && (!new_tokens || !new_src || !n_new || !hidden || hidden_n < 1)) return TLT_EINVAL;
    if (!tree_ok(out_tree) || !out_tree->score || (!root_tokens && !do_extend) || !u_draw || !out_draft_q) return TLT_EINVAL;
    if (B > ctx->max_batch || new_stride > std::max(ctx->max_n, ctx->max_topk)) return TLT_ESHAPE;
    if (depth > ctx->max_depth || topk > ctx->max_topk || n_verify > ctx->max_n) return TLT_ESHAPE;
    // the template and, from it, the work of every level
    int32_t t_parent[TLT_MAX_TREE], t_rank[TLT_MAX_TREE], t_depth[TLT_MAX_TREE], n = 0;
    int rc = tlt_template_build(topk, depth, n_verify, t_parent, t_rank, t_depth, &n);
    if (rc) return rc;
    if (out_tree->n != n) return TLT_EINVAL;
    int first_child[TLT_MAX_TREE], n_child[TLT_MAX_TREE] = {}, inner_idx[TLT_MAX_TREE];
    for (int i = n - 1; i >= 1; --i) {
        first_child[t_parent[i]] = i;   // children are consecutive: the last write is the lowest index
        ++n_child[t_parent[i]];
    }
    int n_inner = 0;   // nodes other than the root that have children = provisional drafter rows
    for (int i = 1; i < n; ++i) inner_idx[i] = n_child[i] ? n_inner++ : -1;
    rc = check_kv(ctx, draft_kv, new_stride + n_inner);
    if (rc) return rc;

    struct DraftFlag {
        tlt_ctx* c;
        explicit DraftFlag(tlt_ctx* x) : c(x) { c->in_draft = true; }
        ~DraftFlag() { c->in_draft = false; }
    } draft_flag(ctx);
    hipStream_t s = (hipStream_t)stream;
    if ((rc = ensure_status(ctx, s))) return rc;
    ctx->pending_parts = 0;
    const tlt_model_cfg& c = ctx->cfg;
    const Plan& p = ctx->plan;
    char* ws = ctx->ws;
    const int h = c.hidden, V = c.vocab, dt = c.dtype;
    const double e = (double)esz_of(ctx);
    float* feat = (float*)(ws + p.feat);
    float* logits = (float*)(ws + p.logits);
    int32_t* fr_token = (int32_t*)(ws + p.fr_token);
    int32_t* fr_src = (int32_t*)(ws + p.fr_src);
    uint64_t* fr_mask = (uint64_t*)(ws + p.fr_mask);
    const int FR = p.feat_rows;
    const tlt_layer_weights& lw = ctx->draft.layers[0];
    KVLayer kvl = kv_layer(ctx, draft_kv, 0);

    if (do_extend && (rc = draft_extend_rows(ctx, s, B, new_tokens, new_src, n_new, new_stride, hidden, hidden_n, draft_kv, kvl)))
        return rc;

    TmplParents tp;
    for (int i = 0; i < TLT_MAX_TREE; ++i) tp.parent[i] = (int8_t)(i < n ? t_parent[i] : -1);
    TLT_RUN(ctx, s, CLS_OTHER, 0, 0,
            tmpl_tree_init(s, B, n, tp, root_tokens, new_tokens, n_new, new_stride, out_tree->token, out_tree->parent,
                           out_tree->score));
    TLT_RUN(ctx, s, CLS_OTHER, 0, 0, tree_finalize(s, B, n, out_tree->parent, out_tree->depth, out_tree->anc_mask));
    if (n == 1) return TLT_OK;

    // the root's distribution (feature row 0 -> final norm -> LM head) and its children
    TmplRows lv;
    lv.R = 1;
    lv.node[0] = 0;
    lv.first_child[0] = (uint8_t)first_child[0];
    lv.n_child[0] = (uint8_t)n_child[0];
    if (!do_extend) {   // (an extend has left it in xn)
        NormIO io;
        io.src_stride = FR;
        TLT_RUN(ctx, s, CLS_OTHER, 0, (double)B * h * (4 + e), rmsnorm(s, dt, B, h, feat, ctx->target.final_norm, c.rms_eps, ws + p.xn, io));
    }
    if ((rc = run_gemm(ctx, s, OUT_F32, B, V, h, ws + p.xn, ctx->target.lm_head, logits))) return rc;
    TLT_RUN(ctx, s, CLS_OTHER, 0, (double)B * V * 12,
            softmax_draw(s, B, n, V, temperature, lv, logits, u_draw, out_tree->token, out_draft_q,
                         ctx->pending_parts == 0 ? ws + p.parts : nullptr, p.parts_bytes));   // (the slices' buffer is idle here)

    // level d: the nodes of depth d that have children, one drafter row each (provisional cache row
    // and feature row 1 + its index among such nodes)
    uint64_t mask_of[TLT_MAX_TREE] = {};
    for (int d = 1; d < depth; ++d) {
        lv.R = 0;
        int slot_base = -1;
        for (int i = 1; i < n; ++i) {
            if (t_depth[i] != d || !n_child[i]) continue;
            const int par = t_parent[i];
            mask_of[i] = (par > 0 ? mask_of[par] : 0ull) | (1ull << inner_idx[i]);
            if (slot_base < 0) slot_base = inner_idx[i];
            const int r = lv.R++;
            lv.node[r] = (uint8_t)i;
            lv.first_child[r] = (uint8_t)first_child[i];
            lv.n_child[r] = (uint8_t)n_child[i];
            lv.src[r] = (uint8_t)(par > 0 ? 1 + inner_idx[par] : 0);
            lv.mask[r] = mask_of[i];
        }
        if (lv.R == 0) break;
        const int M = B * lv.R;
        TLT_RUN(ctx, s, CLS_OTHER, 0, 0, tmpl_level_rows(s, B, n, lv, out_tree->token, fr_token, fr_src, fr_mask));
        TLT_RUN(ctx, s, CLS_OTHER, 0, (double)M * h * (4 + 3 * e),
                draft_input(s, dt, B, lv.R, h, V, fr_token, fr_src, nullptr, FR, (int64_t)B * FR, feat, ctx->target.embed,
                            ws + p.xn));
        if ((rc = draft_fc(ctx, s, M, ws + p.xn))) return rc;
        Rows rows;
        rows.B = B;
        rows.n = lv.R;
        rows.pos_base = d - 1;
        rows.pos_stride = 0;
        rows.slot_base = slot_base;
        rows.mask = fr_mask;
        rows.mask_words = 1;
        rows.n_region = slot_base + lv.R;
        if ((rc = layer_forward(ctx, s, lw, rows, kvl))) return rc;
        NormIO io;
        io.copy = feat;
        io.copy_n = lv.R;
        io.copy_stride = FR;
        io.copy_base = 1 + slot_base;
        if ((rc = norm_lm_head(ctx, s, M, io, logits))) return rc;
        TLT_RUN(ctx, s, CLS_OTHER, 0, (double)M * V * 12,
                softmax_draw(s, B, n, V, temperature, lv, logits, u_draw, out_tree->token, out_draft_q,
                         ctx->pending_parts == 0 ? ws + p.parts : nullptr, p.parts_bytes));   // (the slices' buffer is idle here)
    }
    return TLT_OK;
}

int tlt_accept(tlt_ctx* ctx, void* stream, int B, int mode, float temperature, const tlt_tree* tree,
               const float* target_logits, const int32_t* target_argmax, const float* draft_q, const uint32_t* u_accept,
               const uint32_t* u_final, int stride, int32_t* accept_len, int32_t* path_idx, int32_t* out_tokens,
               int32_t* n_out) {
    if (!ctx || B < 1 || !tree || !tree->token || !tree->parent || tree->n < 1 || tree->n > TLT_MAX_TREE || stride < 1 ||
        !accept_len || !path_idx || !out_tokens || !n_out)
        return TLT_EINVAL;
    if (B > ctx->max_batch || tree->n > ctx->max_n) return TLT_ESHAPE;
    hipStream_t s = (hipStream_t)stream;
    const int n = tree->n, V = ctx->cfg.vocab;
    if (mode == 0) {
        if (!target_argmax && !target_logits) return TLT_EINVAL;
        const int32_t* am = target_argmax;
        if (!am) {
            int32_t* tmp = (int32_t*)(ctx->ws + ctx->plan.argmax);
            TLT_RUN(ctx, s, CLS_OTHER, 0, (double)B * n * V * 4, row_argmax(s, B * n, V, target_logits, tmp));
            am = tmp;
        }
        TLT_RUN(ctx, s, CLS_OTHER, 0, 0,
                accept_greedy(s, B, n, V, stride, tree->token, tree->parent, target_logits, am, accept_len, path_idx,
                              out_tokens, n_out));
        return TLT_OK;
    }
    if (mode == 1) {
        if (!target_logits || !draft_q || !u_accept || !u_final || !(temperature > 0.f)) return TLT_EINVAL;
        int rc = ensure_status(ctx, s);
        if (rc) return rc;
        TLT_RUN(ctx, s, CLS_OTHER, 0, 0,
                accept_sample(s, B, n, V, stride, temperature, tree->token, tree->parent, target_logits, draft_q, u_accept,
                              u_final, accept_len, path_idx, out_tokens, n_out, ctx->ws + ctx->plan.accept_ws,
                              status_word(ctx)));
        return TLT_OK;
    }
    if (mode == 2) {
        if (!target_logits || !u_accept || !u_final || !(temperature > 0.f)) return TLT_EINVAL;
        TLT_RUN(ctx, s, CLS_OTHER, 0, 0,
                accept_target_only(s, B, n, V, stride, temperature, tree->token, tree->parent, target_logits, u_accept,
                                   u_final, accept_len, path_idx, out_tokens, n_out));
        return TLT_OK;
    }
    return TLT_EINVAL;
}

// ---- sampling acceptance on the library's own static scratch (for callers that cannot allocate)
namespace {
constexpr size_t kStaticScratchBytes = (size_t)16 << 20;
constexpr int kMaxDevices = 64;
}  // namespace
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
namespace {
void* g_scratch_ptr[kMaxDevices] = {};   // device address of `scratch` on each GPU (every GPU holds its own copy)

// The array's name is a host-side stand-in, not a device address: the address is asked for once per
// device, with that device current, and only that pointer is handed to kernels.
hipError_t static_scratch(void** out) {
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        e = hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!ptr) return hipErrorInvalidSymbol;
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return hipSuccess;
}
}  // namespace

int tlt_accept_sample_static(void* stream, int B, int vocab, float temperature, const tlt_tree* tree,
                             const float* target_logits, const float* draft_q, const uint32_t* u_accept,
                             const uint32_t* u_final, int stride, int32_t* accept_len, int32_t* path_idx,
                             int32_t* out_tokens, int32_t* n_out, uint32_t* status) {
    if (B < 1 || vocab < 1 || !tree || !tree->token || !tree->parent || tree->n < 1 || tree->n > TLT_MAX_TREE || stride < 1 ||
        !accept_len || !path_idx || !out_tokens || !n_out || !target_logits || !draft_q || !u_accept || !u_final ||
        !(temperature > 0.f))
        return TLT_EINVAL;
    // weights and rendezvous area, then one status word of the library's own (used when the caller passes none)
    const size_t need = accept_sample_workspace_bytes(B, vocab);
    if (need + 256 > kStaticScratchBytes) return TLT_ESHAPE;
    void* ptr = nullptr;
    if (static_scratch(&ptr) != hipSuccess) return TLT_EHIP;
    hipStream_t s = (hipStream_t)stream;
    unsigned int* st = status;
    if (!st) {
        st = (unsigned int*)((char*)ptr + kStaticScratchBytes - 256);
        if (zero_f32(s, 64, (float*)st) != hipSuccess) return TLT_EHIP;
    }
    hipError_t e = accept_sample(s, B, tree->n, vocab, stride, temperature, tree->token, tree->parent, target_logits, draft_q,
                                 u_accept, u_final, accept_len, path_idx, out_tokens, n_out, ptr, st);
    return e == hipSuccess ? TLT_OK : TLT_EHIP;
}

int tlt_kv_commit(tlt_ctx* ctx, void* stream, int B, tlt_kv* kv, const int32_t* accept_len, const int32_t* path_idx,
                  int stride) {
    if (!ctx || B < 1 || !accept_len || !path_idx || stride < 1) return TLT_EINVAL;
    if (!kv || !kv->k_pool || !kv->v_pool || !kv->block_table || !kv->seq_len || kv->n_pages < 1 || kv->max_pages < 1)
        return TLT_EINVAL;
    if (B > ctx->max_batch) return TLT_ESHAPE;
    hipStream_t s = (hipStream_t)stream;
    const tlt_model_cfg& c = ctx->cfg;
    // algorithmic bytes are data dependent (accept lengths live on the device): callers that want
    // a bandwidth figure compute 2 * sum(accept_len) * kv_bytes_per_token themselves
    TLT_RUN(ctx, s, CLS_COMMIT, 0, 0,
            kv_commit(s, c.dtype, B, c.n_layers, kv->k_pool, kv->v_pool, kv->n_pages, kv->block_table, kv->seq_len,
                      kv->max_pages, c.page_size, c.n_kv_heads, c.head_dim, accept_len, path_idx, stride));
    return TLT_OK;
}

size_t tlt_attention_workspace_bytes(int B, int n, int n_q_heads, int n_kv_heads, int head_dim, int max_ctx) {
    if (B < 1 || n < 1 || n > TLT_MAX_TREE || n_q_heads < 1 || n_kv_heads < 1 || n_q_heads % n_kv_heads || max_ctx < 1) return 0;
    return attention_workspace_bytes(B, n, n_q_heads, n_kv_heads, head_dim, max_ctx);
}

int tlt_attention(void* stream, int dtype, int B, int n, int n_q_heads, int n_kv_heads, int head_dim, int page_size,
                  const void* qkv, const uint64_t* anc_mask, const tlt_kv* kv, void* out, void* ws, size_t ws_bytes, int impl) {
    if (B < 1 || n < 1 || n > TLT_MAX_TREE || n_q_heads < 1 || n_kv_heads < 1 || n_q_heads % n_kv_heads || head_dim < 64 ||
        head_dim % 64 || head_dim > 256 || page_size < 1 || (dtype != TLT_F32 && dtype != TLT_BF16) || !qkv || !anc_mask || !out ||
        !ws)
        return TLT_EINVAL;
    if (!kv || !kv->k_pool || !kv->v_pool || !kv->block_table || !kv->seq_len || kv->n_pages < 1 || kv->max_pages < 1 ||
        kv->seq_len_bound < 0)
        return TLT_EINVAL;
    if ((int64_t)kv->seq_len_bound + n > (int64_t)kv->max_pages * page_size) return TLT_ENOPAGES;
    Rows rows;
    rows.B = B;
    rows.n = n;
    rows.mask = anc_mask;
    rows.mask_words = 1;
    rows.n_region = n;
    KVLayer k;
    k.k = kv->k_pool;
    k.v = kv->v_pool;
    k.n_pages = kv->n_pages;
    k.block_table = kv->block_table;
    k.seq_len = kv->seq_len;
    k.max_pages = kv->max_pages;
    k.page_size = page_size;
    k.n_kv = n_kv_heads;
    k.d = head_dim;
    k.seq_len_bound = kv->seq_len_bound;
    hipError_t e = attention((hipStream_t)stream, dtype, rows, k, qkv, out, n_q_heads, ws, ws_bytes, impl);
    return e == hipSuccess ? TLT_OK : (e == hipErrorInvalidValue ? TLT_ESHAPE : TLT_EHIP);
}

int tlt_gemm_glu(void* stream, int M, int N, int K, const void* A, const void* Wg, const void* Wu, void* act) {
    if (M < 1 || N < 1 || K < 1 || !A || !Wg || !Wu || !act) return TLT_EINVAL;
    if (!gemm_glu_supported(TLT_BF16, M, N, K, A, Wg, Wu) || ((uintptr_t)act & 7) != 0) return TLT_ENOTIMPL;   // (8-byte stores)
    return gemm_glu((hipStream_t)stream, TLT_BF16, M, N, K, A, Wg, Wu, act) == hipSuccess ? TLT_OK : TLT_EHIP;
}

int tlt_gemm_parts(void* stream, int M, int N, int K, const void* A, const void* W, float* parts, size_t parts_bytes, int* n_parts) {
    if (M < 1 || N < 1 || K < 1 || !A || !W || !parts || !n_parts || ((uintptr_t)parts & 15) != 0) return TLT_EINVAL;
    if (parts_bytes < (size_t)M * N * 4) return TLT_ESHAPE;
    return gemm_parts((hipStream_t)stream, TLT_BF16, M, N, K, A, W, parts, parts_bytes, n_parts) == hipSuccess ? TLT_OK : TLT_EHIP;
}

int tlt_gemm_argmax(void* stream, int M, int N, int K, const void* A, const void* W, void* ws, size_t ws_bytes,
                    int32_t* out) {
    if (M < 1 || N < 1 || K < 1 || !A || !W || !ws || !out) return TLT_EINVAL;
    if (!gemm_argmax_supported(TLT_BF16, M, N, K, A, W)) return TLT_ENOTIMPL;
    if (ws_bytes < gemm_argmax_workspace_bytes(M, N)) return TLT_ESHAPE;
    return gemm_argmax((hipStream_t)stream, M, N, K, A, W, ws, out) == hipSuccess ? TLT_OK : TLT_EHIP;
}

int tlt_gemm(void* stream, int dtype, int out_mode, int M, int N, int K, const void* A, const void* W, void* C) {
    if (M < 0 || N < 1 || K < 1 || !A || !W || !C || (dtype != TLT_F32 && dtype != TLT_BF16) || out_mode < 0 || out_mode > 2)
        return TLT_EINVAL;
    return gemm((hipStream_t)stream, dtype, out_mode, M, N, K, A, W, C) == hipSuccess ? TLT_OK : TLT_EHIP;
}

int tlt_mfma_stream(void* stream, const void* frags, float* out, int iters) {
    if (!frags || !out || iters < 1 || iters > (1 << 20) || ((uintptr_t)frags & 15) != 0) return TLT_EINVAL;
    return mfma_stream((hipStream_t)stream, frags, out, iters) == hipSuccess ? TLT_OK : TLT_EHIP;
}

int tlt_profile_begin(tlt_ctx* ctx, int enable) {
    if (!ctx) return TLT_EINVAL;
    ctx->prof_on = enable != 0;
    if (enable == 1) ctx->recs.clear();
    return TLT_OK;
}

int tlt_profile_read(tlt_ctx* ctx, double* ms, int64_t* launches, double* flops, double* bytes) {
    if (!ctx || !ms || !launches || !flops || !bytes) return TLT_EINVAL;
    for (int i = 0; i < CLS_N; ++i) {
        ms[i] = 0;
        launches[i] = 0;
        flops[i] = 0;
        bytes[i] = 0;
    }
    for (size_t r = 0; r < ctx->recs.size(); ++r) {
        hipError_t e = hipEventSynchronize(ctx->events[2 * r + 1]);
        if (e != hipSuccess) return fail(ctx, e);
        float t = 0.f;
        e = hipEventElapsedTime(&t, ctx->events[2 * r], ctx->events[2 * r + 1]);
        if (e != hipSuccess) return fail(ctx, e);
        const ProfRec& rec = ctx->recs[r];
        ms[rec.cls] += t;
        launches[rec.cls] += 1;
        flops[rec.cls] += rec.flops;
        bytes[rec.cls] += rec.bytes;
    }
    ctx->recs.clear();
    return TLT_OK;
}


// ---- HIP-graph pool: the greedy step captured per batch bucket, drafter and target apart ------------------
struct tlt_graph_pool {
    tlt_ctx* ctx = nullptr;
    std::vector<int> buckets;
    int bound = 0;                 // sequence-length bound frozen into every graph
    hipStream_t cap = nullptr;     // capture stream (default priority)
    std::map<std::vector<uint64_t>, hipGraphExec_t> draft, target;
    char* snap = nullptr;          // device space for what a warm-up run must not change
    size_t snap_bytes = 0;
};

namespace {

struct Piece {
    void* p;
    size_t bytes;
};

// fn runs once for real on the pool's stream (first-use set-up such as kernel attributes must not fall into a
// capture), the buffers in `keep` get their contents back, and then fn is captured and instantiated.
int capture_graph(tlt_graph_pool* g, const std::vector<Piece>& keep, const std::function<int(hipStream_t)>& fn,
                  hipGraphExec_t* out) {
    tlt_ctx* ctx = g->ctx;
    size_t total = 0;
    for (const Piece& k : keep) total += (k.bytes + 255) & ~(size_t)255;
    hipError_t e;
    if (total > g->snap_bytes) {
        if (g->snap) (void)hipFree(g->snap);
        g->snap = nullptr;
        g->snap_bytes = 0;
        if ((e = hipMalloc((void**)&g->snap, total)) != hipSuccess) return fail(ctx, e);
        g->snap_bytes = total;
    }
    size_t off = 0;
    for (const Piece& k : keep) {
        if ((e = hipMemcpyAsync(g->snap + off, k.p, k.bytes, hipMemcpyDeviceToDevice, g->cap)) != hipSuccess) return fail(ctx, e);
        off += (k.bytes + 255) & ~(size_t)255;
    }
    const bool prof = ctx->prof_on;   // events may not be recorded into a capture
    ctx->prof_on = false;
    int rc = fn(g->cap);
    if (rc == TLT_OK) {
        off = 0;
        for (const Piece& k : keep) {
            if ((e = hipMemcpyAsync(k.p, g->snap + off, k.bytes, hipMemcpyDeviceToDevice, g->cap)) != hipSuccess) rc = fail(ctx, e);
            off += (k.bytes + 255) & ~(size_t)255;
        }
    }
    if (rc == TLT_OK && (e = hipStreamSynchronize(g->cap)) != hipSuccess) rc = fail(ctx, e);
    if (rc == TLT_OK) {
        hipGraph_t graph = nullptr;
        if ((e = hipStreamBeginCapture(g->cap, hipStreamCaptureModeThreadLocal)) != hipSuccess) {
            rc = fail(ctx, e);
        } else {
            rc = fn(g->cap);
            e = hipStreamEndCapture(g->cap, &graph);   // always ends the capture, also after a failed call
            if (rc == TLT_OK && e != hipSuccess) rc = fail(ctx, e);
            if (rc == TLT_OK && (e = hipGraphInstantiate(out, graph, nullptr, nullptr, 0)) != hipSuccess) rc = fail(ctx, e);
            if (graph) (void)hipGraphDestroy(graph);
        }
    }
    ctx->prof_on = prof;
    return rc;
}

void key_kv(std::vector<uint64_t>& k, const tlt_kv* kv) {
    k.push_back((uint64_t)(uintptr_t)kv->k_pool);
    k.push_back((uint64_t)(uintptr_t)kv->v_pool);
    k.push_back((uint64_t)kv->n_pages);
    k.push_back((uint64_t)(uintptr_t)kv->block_table);
    k.push_back((uint64_t)(uintptr_t)kv->seq_len);
    k.push_back((uint64_t)kv->max_pages);
}

void key_tree(std::vector<uint64_t>& k, const tlt_tree* t) {
    k.push_back((uint64_t)(uintptr_t)t->token);
    k.push_back((uint64_t)(uintptr_t)t->parent);
    k.push_back((uint64_t)(uintptr_t)t->depth);
    k.push_back((uint64_t)(uintptr_t)t->anc_mask);
    k.push_back((uint64_t)(uintptr_t)t->score);
    k.push_back((uint64_t)t->n);
}

}  // namespace

int tlt_graph_pool_create(tlt_ctx* ctx, const int32_t* buckets, int n_buckets, int seq_len_bound, tlt_graph_pool** out) {
    if (!ctx || !out || !buckets || n_buckets < 1 || seq_len_bound < 0) return TLT_EINVAL;
    for (int i = 0; i < n_buckets; ++i)
        if (buckets[i] < 1 || buckets[i] > ctx->max_batch || (i > 0 && buckets[i] <= buckets[i - 1])) return TLT_EINVAL;
    tlt_graph_pool* g = new (std::nothrow) tlt_graph_pool();
    if (!g) return TLT_EINVAL;
    g->ctx = ctx;
    g->buckets.assign(buckets, buckets + n_buckets);
    g->bound = seq_len_bound;
    hipError_t e = hipStreamCreateWithFlags(&g->cap, hipStreamNonBlocking);
    if (e != hipSuccess) {
        delete g;
        return fail(ctx, e);
    }
    *out = g;
    return TLT_OK;
}

int tlt_graph_pool_destroy(tlt_graph_pool* g) {
    if (!g) return TLT_OK;
    for (auto& kv : g->draft) (void)hipGraphExecDestroy(kv.second);
    for (auto& kv : g->target) (void)hipGraphExecDestroy(kv.second);
    if (g->snap) (void)hipFree(g->snap);
    if (g->cap) (void)hipStreamDestroy(g->cap);
    delete g;
    return TLT_OK;
}

int tlt_graph_pool_count(const tlt_graph_pool* g, int32_t* n_draft, int32_t* n_target) {
    if (!g || !n_draft || !n_target) return TLT_EINVAL;
    *n_draft = (int32_t)g->draft.size();
    *n_target = (int32_t)g->target.size();
    return TLT_OK;
}

int tlt_graph_pool_step(tlt_graph_pool* g, void* stream, int B, int depth, int topk, int n_verify, const tlt_step_args* a) {
    if (!g || !a || !a->draft_kv || !a->kv || !a->tree || B < 1) return TLT_EINVAL;
    if (!a->new_tokens || !a->new_src || !a->n_new || !a->hidden || !a->argmax || !a->hidden_out || !a->accept_len ||
        !a->path_idx || !a->out_tokens || !a->n_out || a->stride < 1 || a->new_stride < 1 || a->hidden_n < 1)
        return TLT_EINVAL;
    tlt_ctx* ctx = g->ctx;
    int Bk = 0;
    for (int b : g->buckets)
        if (b >= B) {
            Bk = b;
            break;
        }
    if (Bk == 0) return TLT_ESHAPE;
    hipStream_t s = (hipStream_t)stream;
    tlt_kv dkv = *a->draft_kv, kv = *a->kv;
    dkv.seq_len_bound = kv.seq_len_bound = g->bound;
    tlt_tree tree = *a->tree;
    const int h = ctx->cfg.hidden;

    std::vector<uint64_t> dkey = {(uint64_t)Bk, (uint64_t)depth, (uint64_t)topk, (uint64_t)n_verify,
                                  (uint64_t)(uintptr_t)a->new_tokens, (uint64_t)(uintptr_t)a->new_src,
                                  (uint64_t)(uintptr_t)a->n_new, (uint64_t)a->new_stride,
                                  (uint64_t)(uintptr_t)a->hidden, (uint64_t)a->hidden_n};
    key_kv(dkey, &dkv);
    key_tree(dkey, &tree);
    std::vector<uint64_t> tkey = {(uint64_t)Bk, (uint64_t)(uintptr_t)a->argmax, (uint64_t)(uintptr_t)a->hidden_out,
                                  (uint64_t)a->stride, (uint64_t)(uintptr_t)a->accept_len, (uint64_t)(uintptr_t)a->path_idx,
                                  (uint64_t)(uintptr_t)a->out_tokens, (uint64_t)(uintptr_t)a->n_out};
    key_kv(tkey, &kv);
    key_tree(tkey, &tree);

    const bool need_draft = g->draft.find(dkey) == g->draft.end();
    const bool need_target = g->target.find(tkey) == g->target.end();
    if (need_draft || need_target) {
        // captures are rare: everything the caller has queued ends first, so the warm-up runs see its state
        hipError_t e = hipStreamSynchronize(s);
        if (e != hipSuccess) return fail(ctx, e);
    }
    if (need_draft) {
        std::vector<Piece> keep = {{dkv.seq_len, (size_t)Bk * 4}};
        hipGraphExec_t exec = nullptr;
        int rc = capture_graph(g, keep, [&](hipStream_t cs) {
            return tlt_draft_expand(ctx, cs, Bk, depth, topk, n_verify, 0, a->new_tokens, a->new_src, a->n_new, a->new_stride,
                                    a->hidden, a->hidden_n, nullptr, &dkv, &tree);
        }, &exec);
        if (rc != TLT_OK) return rc;
        g->draft[dkey] = exec;
    }
    if (need_target) {
        const size_t row = (size_t)Bk * a->stride * 4;
        std::vector<Piece> keep = {{kv.seq_len, (size_t)Bk * 4}, {a->accept_len, (size_t)Bk * 4}, {a->n_out, (size_t)Bk * 4},
                                   {a->path_idx, row}, {a->out_tokens, row},
                                   {(void*)a->hidden, (size_t)Bk * a->hidden_n * h * 4}};   // hidden_out may be the same buffer
        hipGraphExec_t exec = nullptr;
        int rc = capture_graph(g, keep, [&](hipStream_t cs) {
            int r = tlt_verify_forward(ctx, cs, Bk, &tree, &kv, nullptr, a->argmax, nullptr, a->hidden_out);
            if (r == TLT_OK)
                r = tlt_accept(ctx, cs, Bk, 0, 1.0f, &tree, nullptr, a->argmax, nullptr, nullptr, nullptr, a->stride, a->accept_len,
                               a->path_idx, a->out_tokens, a->n_out);
            if (r == TLT_OK) r = tlt_kv_commit(ctx, cs, Bk, &kv, a->accept_len, a->path_idx, a->stride);
            return r;
        }, &exec);
        if (rc != TLT_OK) return rc;
        g->target[tkey] = exec;
    }
    hipError_t e = hipGraphLaunch(g->draft[dkey], s);
    if (e == hipSuccess) e = hipGraphLaunch(g->target[tkey], s);
    return e == hipSuccess ? TLT_OK : fail(ctx, e);
}

}  // extern "C"
