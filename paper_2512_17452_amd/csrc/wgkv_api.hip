// C ABI of the library: argument checks, host-side bookkeeping, kernel launches.
// Every entry point is documented in include/wgkv.h.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <new>
#include <vector>

#include "wgkv_dev.h"

namespace wgkv {
hipError_t launch_init(const View &pv, hipStream_t st);
hipError_t launch_prefill(const View &pv, const CallSeqs &cs, int layer, float tau, const void *k,
                          const void *v, const float *g, uint8_t *admit_out, int32_t *cnt,
                          int32_t *plan, int nblk_leave_max, int max_T, int max_empty_ring_rows,
                          int max_admitted, hipStream_t st);
hipError_t launch_decode_step(const View &pv, const CallSeqs &cs, int layer, float tau,
                              const void *k, const void *v, const float *g, uint8_t *promoted_out,
                              hipStream_t st);
hipError_t launch_free_seq(const View &pv, int sid, int64_t pages_ub, hipStream_t st);
hipError_t launch_decode_ring(const View &pv, const CallSeqs &cs, int layer, const void *k, const void *v,
                              const float *g, uint8_t *promoted_out, hipStream_t st);
hipError_t launch_decode_promote(const View &pv, const CallSeqs &cs, float tau, hipStream_t st);
hipError_t launch_clear_error(const View &pv, hipStream_t st);
size_t evict_ws_bytes(int n_units);
size_t evict_scores_ws_bytes(const View &pv, int n_units, int n_obs);
hipError_t launch_evict_scores(const View &pv, const CallSeqs &cs, int layer, const void *q_obs, int n_obs,
                               float scale, int pool_w, float *raw, float *out, int64_t stride, int64_t max_len,
                               void *ws, hipStream_t st);
hipError_t launch_evict_apply(const View &pv, const CallSeqs &cs, int layer, const float *scores,
                              int64_t stride, float frac, int32_t *n_evicted, int64_t max_len, hipStream_t st);
size_t quest_landmark_bytes(const View &pv);
hipError_t launch_quest_update(const View &pv, const CallSeqs &cs, int layer, void *landmarks, int reset,
                               hipStream_t st);
hipError_t launch_quest_select(const View &pv, const CallSeqs &cs, int layer, const void *q, void *landmarks,
                               int budget_pages, float *scores, int64_t score_stride, int32_t *sel_pages,
                               int32_t *sel_count, const int32_t *len_ub, hipStream_t st);
size_t attend_decode_ws_bytes(const View &pv, int n_seqs, int grid);
hipError_t static_scratch_init();
void *static_scratch();
hipError_t launch_attend_decode(const View &pv, int layer, int n_seqs, const int32_t *sids,
                                const void *q, float scale, float *out, void *ws, int32_t *counters,
                                int n_cu, int grid_max, hipStream_t st, hipEvent_t ev0, hipEvent_t ev1,
                                const int32_t *sel_pages, const int32_t *sel_count,
                                int sel_stride, int skew_permille);
hipError_t launch_gate_mlp(int dtype, int64_t n_tokens, int n_kv_heads, int head_dim, int width,
                           const void *k, const void *k_rope, const void *w1, const float *b1,
                           const void *w2, const float *b2, float eps, float *g_out, hipStream_t st);
hipError_t launch_gate_linear(int dtype, int64_t n_tokens, int hidden_dim, int n_kv_heads,
                              const void *hidden, const void *w, float *g_out, hipStream_t st);
size_t soft_attn_ws_bytes(int64_t total_tokens, int n_q_heads);
hipError_t launch_soft_attn_fwd(int n_seqs, const int32_t *n_tokens, int Hq, int Hkv, int d, int W,
                                const void *q, const void *k, const void *v, const float *g, float scale,
                                float eps, float *out, float *lse, hipStream_t st);
hipError_t launch_soft_attn_bwd(int n_seqs, const int32_t *n_tokens, int Hq, int Hkv, int d, int W,
                                const void *q, const void *k, const void *v, const float *g, float scale,
                                float eps, const float *out, const float *lse, const void *dout, float *dq,
                                float *dk, float *dv, float *dg, void *ws, hipStream_t st);
size_t sparsity_ws_bytes();
hipError_t launch_sparsity_loss(const float *g, int64_t n, int64_t n_total, float *loss, float *dg, void *ws,
                                hipStream_t st);
hipError_t launch_stream_read(const void *buf, size_t bytes, uint32_t *sink, int n_cu, hipStream_t st,
                              hipEvent_t ev0, hipEvent_t ev1);
size_t attend_prefill_ws_bytes(const View &pv, int n_seqs, int64_t total_q);
size_t attend_prefill_ws_min_bytes();
hipError_t launch_attend_prefill(const View &pv, const CallSeqs &cs, int layer, const void *q,
                                 const void *k, const void *v, const float *g, float tau,
                                 float scale, float *out, void *ws, size_t ws_bytes, int n_cu, hipStream_t st);
hipError_t launch_attend_prefill_f32(const View &pv, const CallSeqs &cs, int layer, const void *q, const void *k,
                                     const void *v, const float *g, float tau, float scale, float *out, void *ws,
                                     size_t ws_bytes, hipStream_t st);
}  // namespace wgkv

using namespace wgkv;

namespace {

constexpr int kPrefillBlkHost = 512;    // must match kPrefillBlk in admit.hip
constexpr int kAttnGridMax = 2048;      // upper bound on the decode-attention grid (blocks of 4 waves)
constexpr int kAttnDefaultSkewPermille = 50;  // see wgkv_tune_decode_attention
constexpr int kAttnStaticGridMax = 512;   // grid bound of the entry point that keeps its partials in the static array

inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

int check_config(const wgkv_config *c) {
    if (!c) return WGKV_ERR_INVALID_ARG;
    if (c->n_layers < 1 || c->n_kv_heads < 1 || c->n_q_heads < 1) return WGKV_ERR_INVALID_ARG;
    if (c->n_q_heads % c->n_kv_heads) return WGKV_ERR_INVALID_ARG;
    const int G = c->n_q_heads / c->n_kv_heads;
    if (G != 1 && G != 2 && G != 4 && G != 8) return WGKV_ERR_INVALID_ARG;
    if (c->head_dim != 64 && c->head_dim != 128) return WGKV_ERR_INVALID_ARG;
    if (c->dtype != WGKV_F32 && c->dtype != WGKV_BF16) return WGKV_ERR_INVALID_ARG;
    if (c->page_size < 1 || (c->page_size & (c->page_size - 1)) || c->page_size > 1024) return WGKV_ERR_INVALID_ARG;
    if (c->w_local < 1 || c->w_local > (1 << 20)) return WGKV_ERR_INVALID_ARG;
    if (c->max_seqs < 1 || c->max_global_pages_per_head < 1) return WGKV_ERR_INVALID_ARG;
    if (c->n_pages < 1 || c->n_pages >= ((int64_t)1 << 31)) return WGKV_ERR_INVALID_ARG;
    const int64_t units = (int64_t)c->max_seqs * c->n_layers * c->n_kv_heads;
    if (units * (int64_t)c->max_global_pages_per_head >= ((int64_t)1 << 40)) return WGKV_ERR_INVALID_ARG;
    return WGKV_OK;
}

void make_layout(const wgkv_config *c, wgkv_meta_layout *o) {
    const size_t S = c->max_seqs, L = c->n_layers, H = c->n_kv_heads;
    const size_t nlp = (c->w_local + c->page_size - 1) / c->page_size;
    size_t off = 0;
    o->seq_len = off;    off = align256(off + S * L * 4);
    o->global_len = off; off = align256(off + S * L * H * 4);
    o->local_pt = off;   off = align256(off + S * L * H * nlp * 4);
    o->global_pt = off;  off = align256(off + S * L * H * (size_t)c->max_global_pages_per_head * 4);
    o->ring_g = off;     off = align256(off + S * L * H * (size_t)c->w_local * 4);
    o->free_stack = off; off = align256(off + (size_t)c->n_pages * 4);
    o->free_top = off;   off = align256(off + 4);
    o->err_flag = off;   off = align256(off + 4);
    o->unit_counters = off; off = align256(off + (size_t)WGKV_MAX_CALL_UNITS * 4);
    o->ahead = off;      off = align256(off + S * L * H * 4);
    o->total_bytes = off;
    o->n_local_pages = (int32_t)nlp;
}

View make_view(const wgkv_config *c, void *pool, void *meta) {
    wgkv_meta_layout lay;
    make_layout(c, &lay);
    View v;
    memset(&v, 0, sizeof(v));
    v.L = c->n_layers; v.Hq = c->n_q_heads; v.Hkv = c->n_kv_heads; v.d = c->head_dim;
    v.dtype = c->dtype; v.es = c->dtype == WGKV_F32 ? 4 : 2;
    v.P = c->page_size; v.logP = 0;
    while ((1 << v.logP) < v.P) v.logP++;
    v.W = c->w_local; v.S = c->max_seqs; v.maxgp = c->max_global_pages_per_head;
    v.nlp = lay.n_local_pages; v.G = c->n_q_heads / c->n_kv_heads;
    v.n_pages = (int32_t)c->n_pages;
    v.row_bytes = (uint32_t)(v.d * v.es);
    v.v_off = (uint32_t)(v.P * v.d * v.es);
    v.page_bytes = (uint64_t)2 * v.P * v.d * v.es;
    v.pool = (char *)pool;
    // a null base (the size query builds a view for its dimensions only) leaves every metadata pointer null
    const auto at = [meta](size_t off) -> void * { return meta ? (char *)meta + off : nullptr; };
    v.seq_len = (int32_t *)at(lay.seq_len);
    v.global_len = (int32_t *)at(lay.global_len);
    v.local_pt = (int32_t *)at(lay.local_pt);
    v.global_pt = (int32_t *)at(lay.global_pt);
    v.ring_g = (float *)at(lay.ring_g);
    v.free_stack = (int32_t *)at(lay.free_stack);
    v.free_top = (int32_t *)at(lay.free_top);
    v.err_flag = (int32_t *)at(lay.err_flag);
    v.unit_counters = (int32_t *)at(lay.unit_counters);
    v.ahead = (int32_t *)at(lay.ahead);
    return v;
}

struct PrefillWs { size_t g_off, cnt_off, plan_off, total; };

// scratch of a prefill call: scores computed from the gate, block counts, plan
PrefillWs prefill_ws(const wgkv_config *c, int n_seqs, int64_t total_tokens, int64_t max_T) {
    PrefillWs w;
    size_t off = 0;
    w.g_off = off;   off = align256(off + (size_t)total_tokens * c->n_kv_heads * 4);
    const size_t n_units = (size_t)n_seqs * c->n_kv_heads;
    const size_t nblk = (size_t)((max_T + kPrefillBlkHost - 1) / kPrefillBlkHost) + 1;
    w.cnt_off = off; off = align256(off + n_units * nblk * 4);
    w.plan_off = off; off = align256(off + (1 + 2 * n_units) * 4);
    w.total = off;
    return w;
}

}  // namespace

struct wgkv_pool {
    wgkv_config cfg;
    View view;
    wgkv_meta_layout lay;
    std::vector<int32_t> seq_len_h;  // [S][L] exact mirror (deterministic)
    std::vector<uint8_t> touched_h;  // [S][L] local pages handed out
    std::vector<int32_t> g_ub;       // [S][L][H] upper bound of the global length
    std::vector<int32_t> ahead_h;    // [S][L] token count whose promotion wgkv_decode_promote has enqueued, else -1
    int64_t pages_ub;                // upper bound of pages in use
    int n_cu;                        // compute units of the device
    int skew_permille;               // decode attention: thousandths of an odd block's tiles given to the even one
    hipEvent_t ev0, ev1;
};

extern "C" {

const char *wgkv_version(void) { return "wgkv-gfx950 0.1"; }

int wgkv_get_meta_layout(const wgkv_config *cfg, wgkv_meta_layout *out) {
    int rc = check_config(cfg);
    if (rc) return rc;
    if (!out) return WGKV_ERR_INVALID_ARG;
    make_layout(cfg, out);
    return WGKV_OK;
}

int wgkv_query_sizes(const wgkv_config *cfg, int32_t max_call_seqs, int64_t max_call_tokens,
                     size_t *pool_bytes, size_t *meta_bytes, size_t *workspace_bytes) {
    int rc = check_config(cfg);
    if (rc) return rc;
    if (max_call_seqs < 1 || max_call_seqs > WGKV_MAX_CALL_SEQS || max_call_tokens < 1 ||
        max_call_tokens >= ((int64_t)1 << 31) ||
        (int64_t)max_call_seqs * cfg->n_kv_heads > WGKV_MAX_CALL_UNITS)
        return WGKV_ERR_INVALID_ARG;
    wgkv_meta_layout lay;
    make_layout(cfg, &lay);
    View v = make_view(cfg, nullptr, nullptr);
    if (pool_bytes) *pool_bytes = (size_t)cfg->n_pages * v.page_bytes;
    if (meta_bytes) *meta_bytes = lay.total_bytes;
    if (workspace_bytes) {
        size_t a = prefill_ws(cfg, max_call_seqs, max_call_tokens, max_call_tokens).total;
        size_t b = attend_decode_ws_bytes(v, max_call_seqs, kAttnGridMax);
        size_t c = attend_prefill_ws_bytes(v, max_call_seqs, max_call_tokens);
        size_t m = a > b ? a : b;
        m = m > c ? m : c;
        size_t e = evict_ws_bytes(max_call_seqs * cfg->n_kv_heads);
        const size_t e2 = evict_scores_ws_bytes(v, max_call_seqs * cfg->n_kv_heads, 256);  // observation windows up to 256
        e = e > e2 ? e : e2;
        *workspace_bytes = align256(m > e ? m : e);
    }
    return WGKV_OK;
}

int wgkv_init_pool(const wgkv_config *cfg, void *pool_dev, size_t pool_bytes, void *meta_dev,
                   size_t meta_bytes, wgkv_stream stream, wgkv_pool **out) {
    int rc = check_config(cfg);
    if (rc) return rc;
    if (!pool_dev || !meta_dev || !out) return WGKV_ERR_INVALID_ARG;
    if (((uintptr_t)pool_dev & 255) || ((uintptr_t)meta_dev & 255)) return WGKV_ERR_INVALID_ARG;
    wgkv_meta_layout lay;
    make_layout(cfg, &lay);
    View v = make_view(cfg, pool_dev, meta_dev);
    if (pool_bytes < (size_t)cfg->n_pages * v.page_bytes || meta_bytes < lay.total_bytes)
        return WGKV_ERR_INVALID_ARG;
    int dev = 0;
    hipDeviceProp_t prop;
    if (hipGetDevice(&dev) != hipSuccess || hipGetDeviceProperties(&prop, dev) != hipSuccess)
        return WGKV_ERR_HIP;
    wgkv_pool *p = new (std::nothrow) wgkv_pool();
    if (!p) return WGKV_ERR_HOST_MEMORY;
    p->cfg = *cfg;
    p->view = v;
    p->lay = lay;
    const size_t n_sl = (size_t)cfg->max_seqs * cfg->n_layers;
    try {
        p->seq_len_h.assign(n_sl, 0);
        p->touched_h.assign(n_sl, 0);
        p->g_ub.assign(n_sl * cfg->n_kv_heads, 0);
        p->ahead_h.assign(n_sl, -1);
    } catch (const std::bad_alloc &) {
        delete p;
        return WGKV_ERR_HOST_MEMORY;
    }
    p->pages_ub = 0;
    p->n_cu = prop.multiProcessorCount > 0 ? prop.multiProcessorCount : 1;
    p->ev0 = p->ev1 = nullptr;
    p->skew_permille = kAttnDefaultSkewPermille;
    // set-up for wgkv_attend_decode_static: this device's address of the static scratch array, so that the call
    // itself asks the runtime nothing
    if (static_scratch_init() != hipSuccess) {
        delete p;
        return WGKV_ERR_HIP;
    }
    if (launch_init(v, (hipStream_t)stream) != hipSuccess) {
        delete p;
        return WGKV_ERR_HIP;
    }
    *out = p;
    return WGKV_OK;
}

void wgkv_destroy(wgkv_pool *pool) { delete pool; }

int wgkv_set_profile_events(wgkv_pool *pool, void *ev_begin, void *ev_end) {
    if (!pool || ((ev_begin == nullptr) != (ev_end == nullptr))) return WGKV_ERR_INVALID_ARG;
    pool->ev0 = (hipEvent_t)ev_begin;
    pool->ev1 = (hipEvent_t)ev_end;
    return WGKV_OK;
}

static int check_seqs(const wgkv_pool *p, int32_t layer, int32_t n_seqs, const int32_t *ids) {
    if (!p || !ids) return WGKV_ERR_INVALID_ARG;
    if (layer < 0 || layer >= p->cfg.n_layers) return WGKV_ERR_INVALID_ARG;
    if (n_seqs < 1 || n_seqs > WGKV_MAX_CALL_SEQS ||
        (int64_t)n_seqs * p->cfg.n_kv_heads > WGKV_MAX_CALL_UNITS)
        return WGKV_ERR_INVALID_ARG;
    for (int i = 0; i < n_seqs; i++) {
        if (ids[i] < 0 || ids[i] >= p->cfg.max_seqs) return WGKV_ERR_INVALID_ARG;
        for (int j = 0; j < i; j++)
            if (ids[j] == ids[i]) return WGKV_ERR_INVALID_ARG;
    }
    return WGKV_OK;
}

int wgkv_gate_scores(int32_t dtype, int64_t n_tokens, int32_t hidden_dim, int32_t n_kv_heads,
                     const void *hidden_dev, const void *gate_w_dev, float *g_out_dev,
                     wgkv_stream stream) {
    if ((dtype != WGKV_F32 && dtype != WGKV_BF16) || n_tokens < 0 || hidden_dim < 8 ||
        (hidden_dim % 8) || n_kv_heads < 1 || n_kv_heads > 16 || !hidden_dev || !gate_w_dev ||
        !g_out_dev || (((uintptr_t)hidden_dev | (uintptr_t)gate_w_dev) & 15) != 0)
        return WGKV_ERR_INVALID_ARG;
    if (n_tokens == 0) return WGKV_OK;
    return launch_gate_linear(dtype, n_tokens, hidden_dim, n_kv_heads, hidden_dev, gate_w_dev,
                              g_out_dev, (hipStream_t)stream) == hipSuccess
               ? WGKV_OK
               : WGKV_ERR_HIP;
}

int wgkv_gate_mlp_scores(int32_t dtype, int64_t n_tokens, int32_t n_kv_heads, int32_t head_dim,
                         int32_t width, const void *k_dev, const void *k_rope_dev,
                         const void *w1_dev, const float *b1_dev, const void *w2_dev,
                         const float *b2_dev, float eps, float *g_out_dev, wgkv_stream stream) {
    if ((dtype != WGKV_F32 && dtype != WGKV_BF16) || n_tokens < 0 || n_kv_heads < 1 ||
        n_kv_heads > 65535 || head_dim < 1 || head_dim > 4096 || width < 1 || !w1_dev || !b1_dev ||
        !w2_dev || !b2_dev || !(eps >= 0.f) || !std::isfinite(eps))
        return WGKV_ERR_INVALID_ARG;
    if (n_tokens == 0) return WGKV_OK;  // nothing to read or write: the token buffers may be NULL
    if (!k_dev || !k_rope_dev || !g_out_dev) return WGKV_ERR_INVALID_ARG;
    if ((((uintptr_t)k_dev | (uintptr_t)k_rope_dev | (uintptr_t)w1_dev) & 15) != 0) return WGKV_ERR_INVALID_ARG;
    return launch_gate_mlp(dtype, n_tokens, n_kv_heads, head_dim, width, k_dev, k_rope_dev, w1_dev,
                           b1_dev, w2_dev, b2_dev, eps, g_out_dev, (hipStream_t)stream) == hipSuccess
               ? WGKV_OK
               : WGKV_ERR_HIP;
}

// Shape and argument checks shared by the two soft-attention entry points; *total gets the rows.
static int soft_attn_check(int32_t dtype, int32_t n_seqs, const int32_t *n_tokens_host, int32_t n_q_heads,
                           int32_t n_kv_heads, int32_t head_dim, int32_t w_local, float scale, float eps,
                           int64_t *total) {
    if (dtype != WGKV_BF16 || head_dim != 128 || n_kv_heads < 1 || n_kv_heads > 65535 ||
        n_q_heads != 4 * n_kv_heads || w_local < 1 || n_seqs < 0 || n_seqs > WGKV_MAX_CALL_SEQS ||
        (n_seqs > 0 && !n_tokens_host) || !std::isfinite(scale) || !(eps >= 0.f) || !std::isfinite(eps))
        return WGKV_ERR_INVALID_ARG;
    int64_t t = 0;
    for (int b = 0; b < n_seqs; b++) {
        if (n_tokens_host[b] < 0) return WGKV_ERR_INVALID_ARG;
        t += n_tokens_host[b];
        if (t >= ((int64_t)1 << 24)) return WGKV_ERR_INVALID_ARG;
    }
    *total = t;
    return WGKV_OK;
}

int wgkv_soft_attn_forward(int32_t dtype, int32_t n_seqs, const int32_t *n_tokens_host,
                           int32_t n_q_heads, int32_t n_kv_heads, int32_t head_dim,
                           int32_t w_local, const void *q_dev, const void *k_dev,
                           const void *v_dev, const float *g_dev, float scale, float eps,
                           float *out_dev, float *lse_dev, wgkv_stream stream) {
    int64_t total = 0;
    int rc = soft_attn_check(dtype, n_seqs, n_tokens_host, n_q_heads, n_kv_heads, head_dim, w_local, scale, eps, &total);
    if (rc) return rc;
    if (total == 0) return WGKV_OK;
    if (!q_dev || !k_dev || !v_dev || !g_dev || !out_dev || !lse_dev) return WGKV_ERR_INVALID_ARG;
    if ((((uintptr_t)q_dev | (uintptr_t)k_dev | (uintptr_t)v_dev | (uintptr_t)out_dev) & 15) != 0)
        return WGKV_ERR_INVALID_ARG;
    return launch_soft_attn_fwd(n_seqs, n_tokens_host, n_q_heads, n_kv_heads, head_dim, w_local, q_dev, k_dev,
                                v_dev, g_dev, scale, eps, out_dev, lse_dev, (hipStream_t)stream) == hipSuccess
               ? WGKV_OK
               : WGKV_ERR_HIP;
}

size_t wgkv_soft_attn_workspace_bytes(int64_t total_tokens, int32_t n_q_heads) {
    if (total_tokens < 0 || n_q_heads < 1) return 0;
    return soft_attn_ws_bytes(total_tokens, n_q_heads);
}

int wgkv_soft_attn_backward(int32_t dtype, int32_t n_seqs, const int32_t *n_tokens_host,
                            int32_t n_q_heads, int32_t n_kv_heads, int32_t head_dim,
                            int32_t w_local, const void *q_dev, const void *k_dev,
                            const void *v_dev, const float *g_dev, float scale, float eps,
                            const float *out_dev, const float *lse_dev, const void *dout_dev,
                            float *dq_dev, float *dk_dev, float *dv_dev, float *dg_dev,
                            void *workspace_dev, size_t workspace_bytes, wgkv_stream stream) {
    int64_t total = 0;
    int rc = soft_attn_check(dtype, n_seqs, n_tokens_host, n_q_heads, n_kv_heads, head_dim, w_local, scale, eps, &total);
    if (rc) return rc;
    if (total == 0) return WGKV_OK;
    if (!q_dev || !k_dev || !v_dev || !g_dev || !out_dev || !lse_dev || !dout_dev || !dq_dev || !dk_dev ||
        !dv_dev || !dg_dev || !workspace_dev)
        return WGKV_ERR_INVALID_ARG;
    if ((((uintptr_t)q_dev | (uintptr_t)k_dev | (uintptr_t)v_dev | (uintptr_t)out_dev | (uintptr_t)dout_dev |
          (uintptr_t)dq_dev | (uintptr_t)dk_dev | (uintptr_t)dv_dev | (uintptr_t)workspace_dev) & 15) != 0)
        return WGKV_ERR_INVALID_ARG;
    if (workspace_bytes < soft_attn_ws_bytes(total, n_q_heads)) return WGKV_ERR_WORKSPACE;
    return launch_soft_attn_bwd(n_seqs, n_tokens_host, n_q_heads, n_kv_heads, head_dim, w_local, q_dev, k_dev,
                                v_dev, g_dev, scale, eps, out_dev, lse_dev, dout_dev, dq_dev, dk_dev, dv_dev,
                                dg_dev, workspace_dev, (hipStream_t)stream) == hipSuccess
               ? WGKV_OK
               : WGKV_ERR_HIP;
}

int wgkv_sparsity_loss(const float *g_dev, int64_t n, int64_t n_total, float *loss_dev, float *dg_dev,
                       void *workspace_dev, size_t workspace_bytes, wgkv_stream stream) {
    if (n < 0 || n_total < 1 || n > n_total || !loss_dev || !workspace_dev || (n > 0 && !g_dev))
        return WGKV_ERR_INVALID_ARG;
    if (workspace_bytes < sparsity_ws_bytes()) return WGKV_ERR_WORKSPACE;
    return launch_sparsity_loss(g_dev, n, n_total, loss_dev, dg_dev, workspace_dev, (hipStream_t)stream) == hipSuccess
               ? WGKV_OK
               : WGKV_ERR_HIP;
}

// max_admitted < 0: no bound from the caller (every leaving token may be admitted)
static int prefill_admit_impl(wgkv_pool *p, int32_t layer, int32_t n_seqs, const int32_t *seq_ids_host,
                              const int32_t *n_tokens_host, const void *k_dev, const void *v_dev,
                              const float *g_dev, const void *hidden_dev, const void *gate_w_dev,
                              int32_t hidden_dim, float tau, int32_t max_admitted, uint8_t *admit_mask_out_dev,
                              void *workspace_dev, size_t workspace_bytes, wgkv_stream stream) {
    int rc = check_seqs(p, layer, n_seqs, seq_ids_host);
    if (rc) return rc;
    if (!n_tokens_host || !workspace_dev) return WGKV_ERR_INVALID_ARG;
    const wgkv_config &c = p->cfg;
    const int W = c.w_local, P = c.page_size, H = c.n_kv_heads;
    CallSeqs cs;
    memset(&cs, 0, sizeof(cs));
    cs.n = n_seqs;
    int64_t total = 0, max_T = 0, max_leave = 0, max_ring = 0;
    for (int b = 0; b < n_seqs; b++) {
        const int T = n_tokens_host[b];
        if (T < 0) return WGKV_ERR_INVALID_ARG;
        const int64_t t0 = p->seq_len_h[(size_t)seq_ids_host[b] * c.n_layers + layer];
        if (t0 + T >= ((int64_t)1 << 30)) return WGKV_ERR_INVALID_ARG;
        // promoted ahead: the victim is in the global cache already and only a decode step may follow
        if (T > 0 && p->ahead_h[(size_t)seq_ids_host[b] * c.n_layers + layer] == t0) return WGKV_ERR_INVALID_ARG;
        cs.sid[b] = seq_ids_host[b];
        cs.t0[b] = (int32_t)t0;
        cs.ntok[b] = T;
        cs.base[b] = (int32_t)total;
        total += T;
        if (total >= ((int64_t)1 << 31) / (H > 0 ? H : 1)) return WGKV_ERR_INVALID_ARG;
        const int64_t leave = std::max<int64_t>(0, t0 + T - W) - std::max<int64_t>(0, t0 - W);
        max_T = std::max<int64_t>(max_T, T);
        max_leave = std::max(max_leave, leave);
        if (t0 < W) max_ring = std::max<int64_t>(max_ring, std::min(T, W));  // ring rows that may go to empty slots
    }
    if (total == 0) return WGKV_OK;
    if (!k_dev || !v_dev) return WGKV_ERR_INVALID_ARG;
    // scores from the linear gate: the same limits as wgkv_gate_scores (at most 16 kv heads, 16-byte rows)
    if (!g_dev && (!hidden_dev || !gate_w_dev || hidden_dim < 8 || (hidden_dim % 8) || H > 16 ||
                   (((uintptr_t)hidden_dev | (uintptr_t)gate_w_dev) & 15) != 0))
        return WGKV_ERR_INVALID_ARG;
    const PrefillWs ws = prefill_ws(&c, n_seqs, total, max_T);
    if (workspace_bytes < ws.total) return WGKV_ERR_WORKSPACE;
    // worst case for the page bounds: every token that leaves the window is admitted, up to the
    // caller's bound per unit if it gave one (the device refuses the call when a unit exceeds it)
    auto admitted_ub = [&](int64_t t0, int T) {
        const int64_t leave = std::max<int64_t>(0, t0 + T - W) - std::max<int64_t>(0, t0 - W);
        return max_admitted >= 0 ? std::min<int64_t>(leave, max_admitted) : leave;
    };
    int64_t new_pages = 0;
    for (int b = 0; b < n_seqs; b++) {
        const int T = cs.ntok[b];
        if (T == 0) continue;
        const size_t sl = (size_t)cs.sid[b] * c.n_layers + layer;
        const int64_t t0 = cs.t0[b];
        const int64_t leave = admitted_ub(t0, T);
        if (!p->touched_h[sl]) new_pages += (int64_t)p->view.nlp * H;
        for (int h = 0; h < H; h++) {
            const int64_t g0 = p->g_ub[sl * H + h], g1 = g0 + leave;
            const int64_t pg1 = (g1 + P - 1) / P;
            if (pg1 > c.max_global_pages_per_head) return WGKV_ERR_PT_OVERFLOW;
            new_pages += pg1 - (g0 + P - 1) / P;
        }
    }
    if (p->pages_ub + new_pages > c.n_pages) return WGKV_ERR_OUT_OF_PAGES;
    hipStream_t st = (hipStream_t)stream;
    char *wsp = (char *)workspace_dev;
    const float *g = g_dev;
    if (!g) {
        float *gw = (float *)(wsp + ws.g_off);
        if (launch_gate_linear(c.dtype, total, hidden_dim, H, hidden_dev, gate_w_dev, gw, st) != hipSuccess)
            return WGKV_ERR_HIP;
        g = gw;
    }
    const int nblk_leave = (int)((max_leave + kPrefillBlkHost - 1) / kPrefillBlkHost);
    if (launch_prefill(p->view, cs, layer, tau, k_dev, v_dev, g, admit_mask_out_dev,
                       (int32_t *)(wsp + ws.cnt_off), (int32_t *)(wsp + ws.plan_off), nblk_leave,
                       (int)max_T, (int)max_ring, max_admitted, st) != hipSuccess)
        return WGKV_ERR_HIP;
    for (int b = 0; b < n_seqs; b++) {
        const int T = cs.ntok[b];
        if (T == 0) continue;
        const size_t sl = (size_t)cs.sid[b] * c.n_layers + layer;
        const int64_t t0 = cs.t0[b];
        const int64_t leave = admitted_ub(t0, T);
        p->touched_h[sl] = 1;
        p->seq_len_h[sl] = (int32_t)(t0 + T);
        for (int h = 0; h < H; h++) p->g_ub[sl * H + h] += (int32_t)leave;
    }
    p->pages_ub += new_pages;
    return WGKV_OK;
}

int wgkv_prefill_admit(wgkv_pool *p, int32_t layer, int32_t n_seqs, const int32_t *seq_ids_host,
                       const int32_t *n_tokens_host, const void *k_dev, const void *v_dev,
                       const float *g_dev, const void *hidden_dev, const void *gate_w_dev,
                       int32_t hidden_dim, float tau, uint8_t *admit_mask_out_dev,
                       void *workspace_dev, size_t workspace_bytes, wgkv_stream stream) {
    return prefill_admit_impl(p, layer, n_seqs, seq_ids_host, n_tokens_host, k_dev, v_dev, g_dev, hidden_dev,
                              gate_w_dev, hidden_dim, tau, -1, admit_mask_out_dev, workspace_dev,
                              workspace_bytes, stream);
}

int wgkv_prefill_admit_bounded(wgkv_pool *p, int32_t layer, int32_t n_seqs, const int32_t *seq_ids_host,
                               const int32_t *n_tokens_host, const void *k_dev, const void *v_dev,
                               const float *g_dev, const void *hidden_dev, const void *gate_w_dev,
                               int32_t hidden_dim, float tau, int32_t max_admitted_per_head,
                               uint8_t *admit_mask_out_dev, void *workspace_dev, size_t workspace_bytes,
                               wgkv_stream stream) {
    if (max_admitted_per_head < 0) return WGKV_ERR_INVALID_ARG;
    return prefill_admit_impl(p, layer, n_seqs, seq_ids_host, n_tokens_host, k_dev, v_dev, g_dev, hidden_dev,
                              gate_w_dev, hidden_dim, tau, max_admitted_per_head, admit_mask_out_dev,
                              workspace_dev, workspace_bytes, stream);
}

int wgkv_decode_step(wgkv_pool *p, int32_t layer, int32_t n_seqs, const int32_t *seq_ids_host,
                     const void *k_new_dev, const void *v_new_dev, const float *g_new_dev,
                     float tau, uint8_t *promoted_out_dev, wgkv_stream stream) {
    int rc = check_seqs(p, layer, n_seqs, seq_ids_host);
    if (rc) return rc;
    if (!k_new_dev || !v_new_dev || !g_new_dev) return WGKV_ERR_INVALID_ARG;
    const wgkv_config &c = p->cfg;
    const int W = c.w_local, P = c.page_size, H = c.n_kv_heads;
    CallSeqs cs;
    memset(&cs, 0, sizeof(cs));
    cs.n = n_seqs;
    int64_t new_pages = 0;
    bool ring_only = true;  // every sequence of the call promoted ahead for this token, ring pages in place
    for (int b = 0; b < n_seqs; b++) {
        const size_t sl = (size_t)seq_ids_host[b] * c.n_layers + layer;
        const int64_t t0 = p->seq_len_h[sl];
        if (t0 + 1 >= ((int64_t)1 << 30)) return WGKV_ERR_INVALID_ARG;
        cs.sid[b] = seq_ids_host[b];
        cs.t0[b] = (int32_t)t0;
        cs.ntok[b] = 1;
        cs.base[b] = b;
        const bool ahead = p->ahead_h[sl] == t0;  // its pages were counted by wgkv_decode_promote
        ring_only = ring_only && ahead && p->touched_h[sl];
        if (!p->touched_h[sl]) new_pages += (int64_t)p->view.nlp * H;
        if (t0 >= W && !ahead)
            for (int h = 0; h < H; h++) {
                const int64_t g0 = p->g_ub[sl * H + h];
                const int64_t pg1 = (g0 + 1 + P - 1) / P;
                if (pg1 > c.max_global_pages_per_head) return WGKV_ERR_PT_OVERFLOW;
                new_pages += pg1 - (g0 + P - 1) / P;
            }
    }
    if (p->pages_ub + new_pages > c.n_pages) return WGKV_ERR_OUT_OF_PAGES;
    const hipError_t e = ring_only ? launch_decode_ring(p->view, cs, layer, k_new_dev, v_new_dev, g_new_dev,
                                                        promoted_out_dev, (hipStream_t)stream)
                                   : launch_decode_step(p->view, cs, layer, tau, k_new_dev, v_new_dev, g_new_dev,
                                                        promoted_out_dev, (hipStream_t)stream);
    if (e != hipSuccess) return WGKV_ERR_HIP;
    for (int b = 0; b < n_seqs; b++) {
        const size_t sl = (size_t)cs.sid[b] * c.n_layers + layer;
        p->touched_h[sl] = 1;
        if (cs.t0[b] >= W && p->ahead_h[sl] != cs.t0[b])
            for (int h = 0; h < H; h++) p->g_ub[sl * H + h] += 1;
        p->seq_len_h[sl] = cs.t0[b] + 1;
    }
    p->pages_ub += new_pages;
    return WGKV_OK;
}

int wgkv_decode_promote(wgkv_pool *p, int32_t n_seqs, const int32_t *seq_ids_host, float tau, wgkv_stream stream) {
    int rc = check_seqs(p, 0, n_seqs, seq_ids_host);
    if (rc) return rc;
    const wgkv_config &c = p->cfg;
    const int W = c.w_local, P = c.page_size, H = c.n_kv_heads, L = c.n_layers;
    CallSeqs cs;
    memset(&cs, 0, sizeof(cs));
    cs.n = n_seqs;
    int64_t new_pages = 0;
    for (int b = 0; b < n_seqs; b++) {
        const size_t sl0 = (size_t)seq_ids_host[b] * L;
        const int64_t t0 = p->seq_len_h[sl0];
        if (t0 + 1 >= ((int64_t)1 << 30)) return WGKV_ERR_INVALID_ARG;
        cs.sid[b] = seq_ids_host[b];
        cs.t0[b] = (int32_t)t0;
        cs.ntok[b] = 1;
        cs.base[b] = b;
        for (int l = 0; l < L; l++) {
            const size_t sl = sl0 + l;
            if (p->seq_len_h[sl] != t0) return WGKV_ERR_INVALID_ARG;  // the layers of a sequence advance together
            if (t0 >= W && p->ahead_h[sl] != t0)
                for (int h = 0; h < H; h++) {
                    const int64_t g0 = p->g_ub[sl * H + h];
                    const int64_t pg1 = (g0 + 1 + P - 1) / P;
                    if (pg1 > c.max_global_pages_per_head) return WGKV_ERR_PT_OVERFLOW;
                    new_pages += pg1 - (g0 + P - 1) / P;
                }
        }
    }
    if (p->pages_ub + new_pages > c.n_pages) return WGKV_ERR_OUT_OF_PAGES;
    if (launch_decode_promote(p->view, cs, tau, (hipStream_t)stream) != hipSuccess) return WGKV_ERR_HIP;
    for (int b = 0; b < n_seqs; b++)
        for (int l = 0; l < L; l++) {
            const size_t sl = (size_t)cs.sid[b] * L + l;
            if (p->ahead_h[sl] == cs.t0[b]) continue;
            if (cs.t0[b] >= W)
                for (int h = 0; h < H; h++) p->g_ub[sl * H + h] += 1;
            p->ahead_h[sl] = cs.t0[b];
        }
    p->pages_ub += new_pages;
    return WGKV_OK;
}

int wgkv_attend(wgkv_pool *p, int32_t layer, int32_t n_seqs, const int32_t *seq_ids_host,
                const int32_t *n_q_host, const void *q_dev, const void *k_chunk_dev,
                const void *v_chunk_dev, const float *g_chunk_dev, float tau, float scale,
                float *out_dev, void *workspace_dev, size_t workspace_bytes, wgkv_stream stream) {
    int rc = check_seqs(p, layer, n_seqs, seq_ids_host);
    if (rc) return rc;
    if (!n_q_host || !q_dev || !out_dev || !workspace_dev || !std::isfinite(scale)) return WGKV_ERR_INVALID_ARG;
    if ((((uintptr_t)q_dev | (uintptr_t)out_dev | (uintptr_t)workspace_dev) & 15) != 0) return WGKV_ERR_INVALID_ARG;
    const bool prefill = k_chunk_dev != nullptr;
    if (prefill != (v_chunk_dev != nullptr) || prefill != (g_chunk_dev != nullptr)) return WGKV_ERR_INVALID_ARG;
    hipStream_t st = (hipStream_t)stream;
    if (!prefill) {
        for (int b = 0; b < n_seqs; b++)
            if (n_q_host[b] != 1) return WGKV_ERR_INVALID_ARG;
        if (workspace_bytes < attend_decode_ws_bytes(p->view, n_seqs, kAttnGridMax)) return WGKV_ERR_WORKSPACE;
        return launch_attend_decode(p->view, layer, n_seqs, seq_ids_host, q_dev, scale, out_dev,
                                    workspace_dev, p->view.unit_counters, p->n_cu, kAttnGridMax, st, p->ev0, p->ev1, nullptr, nullptr,
                                    0, p->skew_permille) == hipSuccess
                   ? WGKV_OK
                   : WGKV_ERR_HIP;
    }
    if ((((uintptr_t)k_chunk_dev | (uintptr_t)v_chunk_dev) & 15) != 0) return WGKV_ERR_INVALID_ARG;
    CallSeqs cs;
    memset(&cs, 0, sizeof(cs));
    cs.n = n_seqs;
    int64_t total = 0;
    for (int b = 0; b < n_seqs; b++) {
        if (n_q_host[b] < 0) return WGKV_ERR_INVALID_ARG;
        cs.sid[b] = seq_ids_host[b];
        cs.t0[b] = p->seq_len_h[(size_t)seq_ids_host[b] * p->cfg.n_layers + layer];
        cs.ntok[b] = n_q_host[b];
        cs.base[b] = (int32_t)total;
        total += n_q_host[b];
        if (total >= ((int64_t)1 << 31) / p->cfg.n_q_heads) return WGKV_ERR_INVALID_ARG;
    }
    if (total == 0) return WGKV_OK;
    if (workspace_bytes < attend_prefill_ws_min_bytes()) return WGKV_ERR_WORKSPACE;  // what is more holds the picked keys
    if (p->ev0 && hipEventRecord(p->ev0, st) != hipSuccess) return WGKV_ERR_HIP;
    const hipError_t e = p->cfg.dtype == WGKV_BF16
                             ? launch_attend_prefill(p->view, cs, layer, q_dev, k_chunk_dev, v_chunk_dev, g_chunk_dev,
                                                     tau, scale, out_dev, workspace_dev, workspace_bytes, p->n_cu, st)
                             : launch_attend_prefill_f32(p->view, cs, layer, q_dev, k_chunk_dev, v_chunk_dev,
                                                         g_chunk_dev, tau, scale, out_dev, workspace_dev, workspace_bytes,
                                                         st);
    if (e != hipSuccess) return WGKV_ERR_HIP;
    if (p->ev1 && hipEventRecord(p->ev1, st) != hipSuccess) return WGKV_ERR_HIP;
    return WGKV_OK;
}

int wgkv_attend_decode_static(wgkv_pool *p, int32_t layer, int32_t n_seqs, const int32_t *seq_ids_host,
                              const void *q_dev, float scale, float *out_dev, wgkv_stream stream) {
    int rc = check_seqs(p, layer, n_seqs, seq_ids_host);
    if (rc) return rc;
    if (!q_dev || !out_dev || !std::isfinite(scale)) return WGKV_ERR_INVALID_ARG;
    if ((((uintptr_t)q_dev | (uintptr_t)out_dev) & 15) != 0) return WGKV_ERR_INVALID_ARG;
    if (attend_decode_ws_bytes(p->view, n_seqs, kAttnStaticGridMax) > (size_t)WGKV_STATIC_SCRATCH_BYTES)
        return WGKV_ERR_WORKSPACE;  // the call is larger than the static array: use wgkv_attend
    void *ws = static_scratch();
    if (!ws) return WGKV_ERR_HIP;  // no pool was ever initialised on the current device
    return launch_attend_decode(p->view, layer, n_seqs, seq_ids_host, q_dev, scale, out_dev, ws,
                                p->view.unit_counters, p->n_cu, kAttnStaticGridMax,
                                (hipStream_t)stream, p->ev0, p->ev1, nullptr, nullptr, 0, p->skew_permille) == hipSuccess
               ? WGKV_OK
               : WGKV_ERR_HIP;
}

int wgkv_quest_landmark_bytes(const wgkv_config *cfg, size_t *landmark_bytes) {
    int rc = check_config(cfg);
    if (rc) return rc;
    if (!landmark_bytes) return WGKV_ERR_INVALID_ARG;
    View v = make_view(cfg, nullptr, nullptr);
    *landmark_bytes = quest_landmark_bytes(v);
    return WGKV_OK;
}

static int quest_seqs(wgkv_pool *p, int32_t layer, int32_t n_seqs, const int32_t *seq_ids_host, CallSeqs *cs,
                      int64_t *max_len) {
    int rc = check_seqs(p, layer, n_seqs, seq_ids_host);
    if (rc) return rc;
    memset(cs, 0, sizeof(*cs));
    cs->n = n_seqs;
    *max_len = 0;
    const int H = p->cfg.n_kv_heads;
    for (int b = 0; b < n_seqs; b++) {
        const size_t sl = (size_t)seq_ids_host[b] * p->cfg.n_layers + layer;
        cs->sid[b] = seq_ids_host[b];
        cs->t0[b] = p->seq_len_h[sl];
        for (int h = 0; h < H; h++) *max_len = *max_len > p->g_ub[sl * H + h] ? *max_len : p->g_ub[sl * H + h];
    }
    return WGKV_OK;
}

int wgkv_quest_update(wgkv_pool *p, int32_t layer, int32_t n_seqs, const int32_t *seq_ids_host,
                      void *landmarks_dev, size_t landmark_bytes, int32_t reset, wgkv_stream stream) {
    CallSeqs cs;
    int64_t max_len;
    int rc = quest_seqs(p, layer, n_seqs, seq_ids_host, &cs, &max_len);
    if (rc) return rc;
    if (!landmarks_dev || landmark_bytes < quest_landmark_bytes(p->view) || ((uintptr_t)landmarks_dev & 15) != 0)
        return WGKV_ERR_INVALID_ARG;
    return launch_quest_update(p->view, cs, layer, landmarks_dev, reset != 0, (hipStream_t)stream) == hipSuccess
               ? WGKV_OK
               : WGKV_ERR_HIP;
}

int wgkv_quest_select(wgkv_pool *p, int32_t layer, int32_t n_seqs, const int32_t *seq_ids_host,
                      const void *q_dev, void *landmarks_dev, size_t landmark_bytes, int32_t budget_pages,
                      float *page_scores_out_dev, int64_t score_stride, int32_t *sel_pages_out_dev,
                      int32_t *sel_count_out_dev, wgkv_stream stream) {
    CallSeqs cs;
    int64_t max_len;
    int rc = quest_seqs(p, layer, n_seqs, seq_ids_host, &cs, &max_len);
    if (rc) return rc;
    const int P = p->cfg.page_size;
    const int64_t max_pages = (max_len + P - 1) / P;
    if (!q_dev || !landmarks_dev || landmark_bytes < quest_landmark_bytes(p->view) || budget_pages < 1 ||
        !page_scores_out_dev || score_stride < max_pages || !sel_pages_out_dev || !sel_count_out_dev ||
        (((uintptr_t)q_dev | (uintptr_t)landmarks_dev) & 15) != 0)  // both are read 16 bytes per lane
        return WGKV_ERR_INVALID_ARG;
    int32_t len_ub[WGKV_MAX_CALL_UNITS];  // the host's bounds of the heads' lengths, in the call's unit order
    const int H = p->cfg.n_kv_heads;
    for (int b = 0; b < n_seqs; b++)
        for (int h = 0; h < H; h++)
            len_ub[b * H + h] = p->g_ub[((size_t)seq_ids_host[b] * p->cfg.n_layers + layer) * H + h];
    return launch_quest_select(p->view, cs, layer, q_dev, landmarks_dev, budget_pages, page_scores_out_dev,
                               score_stride, sel_pages_out_dev, sel_count_out_dev, len_ub,
                               (hipStream_t)stream) == hipSuccess
               ? WGKV_OK
               : WGKV_ERR_HIP;
}

int wgkv_attend_selected(wgkv_pool *p, int32_t layer, int32_t n_seqs, const int32_t *seq_ids_host,
                         const void *q_dev, const int32_t *sel_pages_dev, const int32_t *sel_count_dev,
                         int32_t sel_stride, float scale, float *out_dev, void *workspace_dev,
                         size_t workspace_bytes, wgkv_stream stream) {
    int rc = check_seqs(p, layer, n_seqs, seq_ids_host);
    if (rc) return rc;
    if (!q_dev || !sel_pages_dev || !sel_count_dev || sel_stride < 1 || !out_dev || !workspace_dev ||
        !std::isfinite(scale))
        return WGKV_ERR_INVALID_ARG;
    if (workspace_bytes < attend_decode_ws_bytes(p->view, n_seqs, kAttnGridMax)) return WGKV_ERR_WORKSPACE;
    return launch_attend_decode(p->view, layer, n_seqs, seq_ids_host, q_dev, scale, out_dev, workspace_dev,
                                p->view.unit_counters, p->n_cu, kAttnGridMax,
                                (hipStream_t)stream, p->ev0, p->ev1, sel_pages_dev, sel_count_dev, sel_stride,
                                p->skew_permille) == hipSuccess
               ? WGKV_OK
               : WGKV_ERR_HIP;
}

int wgkv_evict_scores(wgkv_pool *p, int32_t layer, int32_t n_seqs, const int32_t *seq_ids_host,
                      const void *q_obs_dev, int32_t n_obs, float scale, int32_t pool_w,
                      float *scores_raw_out_dev, float *scores_out_dev, int64_t stride,
                      void *workspace_dev, size_t workspace_bytes, wgkv_stream stream) {
    int rc = check_seqs(p, layer, n_seqs, seq_ids_host);
    if (rc) return rc;
    if (!q_obs_dev || !scores_raw_out_dev || !scores_out_dev || scores_raw_out_dev == scores_out_dev ||
        !workspace_dev || n_obs < 1 || n_obs > 4096 || pool_w < 1 || pool_w > 255 || pool_w % 2 == 0 ||
        !std::isfinite(scale) || stride < 0 || 64 % p->view.G != 0)
        return WGKV_ERR_INVALID_ARG;
    const wgkv_config &c = p->cfg;
    const int H = c.n_kv_heads;
    if (workspace_bytes < evict_scores_ws_bytes(p->view, n_seqs * H, n_obs)) return WGKV_ERR_WORKSPACE;
    CallSeqs cs;
    memset(&cs, 0, sizeof(cs));
    cs.n = n_seqs;
    int64_t max_len = 0;
    for (int b = 0; b < n_seqs; b++) {
        const size_t sl = (size_t)seq_ids_host[b] * c.n_layers + layer;
        cs.sid[b] = seq_ids_host[b];
        cs.t0[b] = p->seq_len_h[sl];
        for (int h = 0; h < H; h++) {
            if (p->g_ub[sl * H + h] > stride) return WGKV_ERR_INVALID_ARG;  // a row must cover what a head may hold
            max_len = max_len > p->g_ub[sl * H + h] ? max_len : p->g_ub[sl * H + h];
        }
    }
    return launch_evict_scores(p->view, cs, layer, q_obs_dev, n_obs, scale, pool_w, scores_raw_out_dev,
                               scores_out_dev, stride, max_len, workspace_dev,
                               (hipStream_t)stream) == hipSuccess
               ? WGKV_OK
               : WGKV_ERR_HIP;
}

int wgkv_evict_apply(wgkv_pool *p, int32_t layer, int32_t n_seqs, const int32_t *seq_ids_host,
                     const float *scores_dev, int64_t stride, float frac,
                     int32_t *n_evicted_out_dev, void *workspace_dev, size_t workspace_bytes,
                     wgkv_stream stream) {
    int rc = check_seqs(p, layer, n_seqs, seq_ids_host);
    if (rc) return rc;
    if (!scores_dev || !workspace_dev || !(frac >= 0.f) || !(frac <= 1.f) || stride < 0)
        return WGKV_ERR_INVALID_ARG;
    const wgkv_config &c = p->cfg;
    const int H = c.n_kv_heads, P = c.page_size;
    if (workspace_bytes < evict_ws_bytes(n_seqs * H)) return WGKV_ERR_WORKSPACE;
    CallSeqs cs;
    memset(&cs, 0, sizeof(cs));
    cs.n = n_seqs;
    int64_t max_len = 0;
    for (int b = 0; b < n_seqs; b++) {
        const size_t sl = (size_t)seq_ids_host[b] * c.n_layers + layer;
        cs.sid[b] = seq_ids_host[b];
        cs.t0[b] = p->seq_len_h[sl];
        // a score row must cover every entry the head may hold (the host knows an upper bound)
        for (int h = 0; h < H; h++) {
            if (p->g_ub[sl * H + h] > stride) return WGKV_ERR_INVALID_ARG;
            max_len = std::max<int64_t>(max_len, p->g_ub[sl * H + h]);
        }
    }
    if (launch_evict_apply(p->view, cs, layer, scores_dev, stride, frac, n_evicted_out_dev, max_len,
                           (hipStream_t)stream) != hipSuccess)
        return WGKV_ERR_HIP;
    // bounds after the call: N - floor(frac N) does not decrease with N, so it maps an upper
    // bound of the length to an upper bound of the new length
    for (int b = 0; b < n_seqs; b++) {
        const size_t sl = (size_t)seq_ids_host[b] * c.n_layers + layer;
        for (int h = 0; h < H; h++) {
            const int64_t g0 = p->g_ub[sl * H + h];
            const int64_t g1 = g0 - (int64_t)floor((double)frac * (double)g0);
            p->pages_ub -= (g0 + P - 1) / P - (g1 + P - 1) / P;
            p->g_ub[sl * H + h] = g1;
        }
    }
    return WGKV_OK;
}

int wgkv_tune_decode_attention(wgkv_pool *p, int32_t n_seqs, const int32_t *seq_ids_host, const void *q_dev,
                               float scale, float *out_dev, void *workspace_dev, size_t workspace_bytes,
                               wgkv_stream stream, int32_t *skew_permille_out) {
    int rc = check_seqs(p, 0, n_seqs, seq_ids_host);
    if (rc) return rc;
    if (!q_dev || !out_dev || !workspace_dev || !std::isfinite(scale)) return WGKV_ERR_INVALID_ARG;
    if ((((uintptr_t)q_dev | (uintptr_t)out_dev | (uintptr_t)workspace_dev) & 15) != 0) return WGKV_ERR_INVALID_ARG;
    if (workspace_bytes < attend_decode_ws_bytes(p->view, n_seqs, kAttnGridMax)) return WGKV_ERR_WORKSPACE;
    hipStream_t st = (hipStream_t)stream;
    static constexpr int kCand[] = {0, 25, 50, 75, 100, 125};
    constexpr int kNc = (int)(sizeof(kCand) / sizeof(kCand[0])), kReps = 5;
    const int L = p->cfg.n_layers;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    if (hipEventCreate(&e0) != hipSuccess) return WGKV_ERR_HIP;
    if (hipEventCreate(&e1) != hipSuccess) { (void)hipEventDestroy(e0); return WGKV_ERR_HIP; }
    float ms_of[kNc][kReps];
    bool ok = true;
    // One measurement of a candidate is a pass over all layers, as a decode step makes it (a layer that is
    // read again right away would come out of the memory-side cache in part); the candidates in turn, several
    // times over, the first time to warm up.  Launches of one kernel on one state: only the split differs.
    for (int r = 0; r < kReps + 1 && ok; r++)
        for (int c = 0; c < kNc && ok; c++) {
            float sum = 0.f;
            for (int l = 0; l < L && ok; l++) {
                ok = launch_attend_decode(p->view, l, n_seqs, seq_ids_host, q_dev, scale, out_dev, workspace_dev,
                                          p->view.unit_counters, p->n_cu, kAttnGridMax, st, e0,
                                          e1, nullptr, nullptr, 0, kCand[c]) == hipSuccess &&
                     hipEventSynchronize(e1) == hipSuccess;
                float ms = 0.f;
                ok = ok && hipEventElapsedTime(&ms, e0, e1) == hipSuccess;
                sum += ms;
            }
            if (ok && r > 0) ms_of[c][r - 1] = sum;
        }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    if (!ok) return WGKV_ERR_HIP;
    float med[kNc];
    for (int c = 0; c < kNc; c++) {
        std::sort(ms_of[c], ms_of[c] + kReps);
        med[c] = ms_of[c][kReps / 2];
    }
    int best = 0;
    for (int c = 1; c < kNc; c++)
        if (med[c] < med[best]) best = c;
    // the default stays unless something else is clearly (one per cent) better: a tuned value changes the
    // rounding of the outputs, and noise should not
    const int def = 2;
    static_assert(kCand[2] == kAttnDefaultSkewPermille, "the default is one of the candidates");
    if (med[best] > 0.99f * med[def]) best = def;
    p->skew_permille = kCand[best];
    if (skew_permille_out) *skew_permille_out = kCand[best];
    return WGKV_OK;
}

int wgkv_free_seq(wgkv_pool *p, int32_t seq_id, wgkv_stream stream) {
    if (!p || seq_id < 0 || seq_id >= p->cfg.max_seqs) return WGKV_ERR_INVALID_ARG;
    const wgkv_config &c = p->cfg;
    const int P = c.page_size, H = c.n_kv_heads;
    int64_t pages = 0;
    for (int l = 0; l < c.n_layers; l++) {
        const size_t sl = (size_t)seq_id * c.n_layers + l;
        if (p->touched_h[sl]) pages += (int64_t)p->view.nlp * H;
        for (int h = 0; h < H; h++) pages += (p->g_ub[sl * H + h] + P - 1) / P;
    }
    if (launch_free_seq(p->view, seq_id, pages, (hipStream_t)stream) != hipSuccess) return WGKV_ERR_HIP;
    p->pages_ub -= pages;
    for (int l = 0; l < c.n_layers; l++) {
        const size_t sl = (size_t)seq_id * c.n_layers + l;
        for (int h = 0; h < H; h++) p->g_ub[sl * H + h] = 0;
        p->touched_h[sl] = 0;
        p->seq_len_h[sl] = 0;
        p->ahead_h[sl] = -1;
    }
    return WGKV_OK;
}

int wgkv_status(wgkv_pool *p, wgkv_stream stream, int64_t *pages_free, int32_t *device_error_flag) {
    if (!p) return WGKV_ERR_INVALID_ARG;
    hipStream_t st = (hipStream_t)stream;
    int32_t top = 0, flag = 0;
    std::vector<int32_t> gl(p->g_ub.size()), sl_dev(p->seq_len_h.size());
    if (hipMemcpyAsync(&top, p->view.free_top, 4, hipMemcpyDeviceToHost, st) != hipSuccess ||
        hipMemcpyAsync(&flag, p->view.err_flag, 4, hipMemcpyDeviceToHost, st) != hipSuccess ||
        hipMemcpyAsync(gl.data(), p->view.global_len, gl.size() * 4, hipMemcpyDeviceToHost, st) != hipSuccess ||
        hipMemcpyAsync(sl_dev.data(), p->view.seq_len, sl_dev.size() * 4, hipMemcpyDeviceToHost, st) != hipSuccess ||
        hipStreamSynchronize(st) != hipSuccess)
        return WGKV_ERR_HIP;
    if (pages_free) *pages_free = top;
    if (device_error_flag) *device_error_flag = flag;
    const wgkv_config &c = p->cfg;
    int64_t used = 0;
    for (size_t sl = 0; sl < p->touched_h.size(); sl++) {
        // token counts as the device has them: replays of a captured decode step advance them
        // without the host seeing it
        p->seq_len_h[sl] = sl_dev[sl];
        p->ahead_h[sl] = -1;  // unknown from here: the full decode step looks at the device's stamps itself
        p->touched_h[sl] = sl_dev[sl] > 0;
        if (p->touched_h[sl]) used += (int64_t)p->view.nlp * c.n_kv_heads;
        for (int h = 0; h < c.n_kv_heads; h++) {
            const size_t i = sl * c.n_kv_heads + h;
            p->g_ub[i] = gl[i];
            used += (gl[i] + c.page_size - 1) / c.page_size;
        }
    }
    p->pages_ub = used;
    // the mirrors are exact again whatever the flag says: a call that set it changed nothing
    return flag != 0 ? WGKV_ERR_DEVICE_FLAG : WGKV_OK;
}

int wgkv_stream_read_probe(const void *buf_dev, size_t bytes, uint32_t *sink_dev, void *ev_begin, void *ev_end,
                           wgkv_stream stream) {
    if (!buf_dev || !sink_dev || bytes < 16 || ((uintptr_t)buf_dev & 15) || ((ev_begin == nullptr) != (ev_end == nullptr)))
        return WGKV_ERR_INVALID_ARG;
    int dev = 0, n_cu = 0;
    if (hipGetDevice(&dev) != hipSuccess ||
        hipDeviceGetAttribute(&n_cu, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n_cu < 1)
        return WGKV_ERR_HIP;
    return launch_stream_read(buf_dev, bytes, sink_dev, n_cu, (hipStream_t)stream, (hipEvent_t)ev_begin,
                              (hipEvent_t)ev_end) == hipSuccess
               ? WGKV_OK
               : WGKV_ERR_HIP;
}

int wgkv_clear_error(wgkv_pool *p, wgkv_stream stream) {
    if (!p) return WGKV_ERR_INVALID_ARG;
    return launch_clear_error(p->view, (hipStream_t)stream) == hipSuccess ? WGKV_OK : WGKV_ERR_HIP;
}

}  // extern "C"
