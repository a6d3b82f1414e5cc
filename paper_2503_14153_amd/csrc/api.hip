// Host side of libspecdec: handle management, argument validation, and the sequencing of the
// kernels of one speculative step (paper Section III-B) on a caller-supplied HIP stream.
#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <new>
#include <vector>

#include "sd_internal.h"
#include "attn_geom.h"

// ------------------------------------------------------------------------------------------ errors
static thread_local char g_err[512] = "";

static int fail(int code, const char* fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof(g_err), fmt, ap);
    va_end(ap);
    return code;
}
#define HIP_TRY(expr)                                                                              \
    do {                                                                                           \
        hipError_t e_ = (expr);                                                                    \
        if (e_ != hipSuccess) return fail(SD_ERR_HIP, "%s: %s", #expr, hipGetErrorString(e_));     \
    } while (0)

extern "C" const char* sd_last_error(void) { return g_err; }
extern "C" const char* sd_version(void) { return "libspecdec 0.1 (gfx950)"; }

static inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }
static inline int ceil_div(int a, int b) { return (a + b - 1) / b; }
static inline int pow2_blocks(int rows);
static inline int prompt_blocks(int rows) { return rows <= 256 ? pow2_blocks(rows) : ceil_div(rows, 32); }   // of a prompt pass
static inline int pow2_blocks(int rows) {   // 32-row blocks, rounded up to 1, 2, 4 or 8
    int mb = ceil_div(rows, 32), p = 1;
    while (p < mb) p *= 2;
    return p;
}

// ------------------------------------------------------------------------------------------ handles
struct LayerW {
    const void *attn_norm, *ffn_norm;       // bf16 [d]
    const void *wqkv, *wo, *wgu, *wdown;    // packed fragments
};

// Optional per-launch timing of the two bandwidth-bound kernel classes with HIP events on the
// caller's stream (sd_profile_begin / sd_profile_end).
enum { KW_QKV, KW_O, KW_DOWN };      // sd_model::kw
enum { PROF_GEMM = 0, PROF_ATTN = 1, PROF_CLASSES = 2 };
struct Profile {
    bool on = false;
    std::vector<hipEvent_t> ev;              // pairs (start, stop)
    std::vector<int> cls;                    // class of pair i
    std::vector<double> bytes;               // algorithmic bytes of pair i
    size_t used = 0;                         // pairs used
};

// What a pass leaves in the tree K/V scratch: its cache's batch, padded rows per sequence, and the sequences that it holds,
// in order, each with its own rows (tree nodes, prompt tokens); float32: the rows of the pass and every sequence's first.
struct ScratchRows {
    int B = 0, Tp = 0, M = 0, n = 0;
    int seq[SD_MAX_BATCH] = {}, len[SD_MAX_BATCH] = {};
    SeqList row0 = {};
};

// Prompt passes of more than 256 rows: packed rows at most, and rows padded to [chunk][Tp] at most.
#define PROMPT_ROWS 1024
#define PROMPT_PADDED 2048

struct sd_model {
    sd_config cfg;
    Profile prof;
    int max_rows, MBmax;
    int KBd, KBf, Fpad, NBqkv, NBo, NBgu, NBv, Vpad, NBmed;
    char* arena = nullptr;                   // packed weights
    char* work = nullptr;                    // workspace
    const void *embed, *lm_head, *final_norm, *medusa_w;
    MedusaBias medusa_b;
    std::vector<LayerW> layers;
    // workspace
    float *x, *part, *logits, *hlogits, *hf, *h_rows, *opart;
    float2* mlpart;
    void *xn, *attn_x, *act, *q, *kt, *vt;
    void* xh;                                // draft-head rows of every tree row, in 256-row operand chunks
    int draft_schedule = SD_DRAFT_AFTER_ACCEPT;
    RowTable rt;
    double* rope_freq;                       // [head_dim / 2]
    PassMap* rm_dev;                         // the row map of a prompt pass, in device memory
    int prompt_rows = 0;                     // rows of the largest prompt pass; above 256 its plans and buffers exist:
    KwPlan kw[2][3];                         // 16, 32 rows; QKV, O, down projection
    std::vector<GemmPlan> prompt_plans;      // of 9 .. prompt_rows / 32 row blocks
    std::vector<double> prompt_us;           // [row blocks]: modelled time of a layer of a pass of that many
    void *ktp = nullptr, *vtp = nullptr;     // one layer's keys and values of such a pass, [chunk][head][blocks]
    int32_t *g_parent, *g_depth, *g_rank, *fin_rows;
    float2* best; void* ranked;                 // ranking scratch: arg-max per row and chunk, top-k per head row and chunk
    float4* row_stats;                     // [Mp]: per tree row, statistics for typical acceptance
    uint32_t* zero_stop;
    const void* zfrag;                       // 2 KiB of zeros
    size_t part_floats;
    int max_parts;
    // HIP-graph mode: one captured graph per distinct launch sequence of a step
    struct StepGraph { std::vector<uint64_t> key; hipGraphExec_t exec; };
    bool use_graphs = false;
    std::vector<StepGraph> graphs;
    hipStream_t cap_stream = nullptr;      // capture happens here: the caller's stream may be the null stream
    std::vector<GemmPlan> plans;             // one per (row blocks, K blocks, N blocks) in use
    int32_t* plan_cnt = nullptr;             // device: the plans' per-group slot counts
    // every shape a call can issue is planned at creation; the entry points check the plans they need
    // (have_plans) before they enqueue anything, so a miss here cannot happen after that check
    const GemmPlan* find_plan(int MB, int KB, int NB) const {
        for (const GemmPlan& p : plans)
            if (p.MB == MB && p.KB == KB && p.NB == NB) return &p;
        for (const GemmPlan& p : prompt_plans)
            if (p.MB == MB && p.KB == KB && p.NB == NB) return &p;
        return nullptr;
    }
    // persistent layer kernel (fused.hip)
    bool fused_ok = false;                   // the device holds its 256 workgroups at once and the buffers exist
    bool use_fused = false;                  // sd_set_fused
    bool fused_dirty = false;                // launched since the host last looked at the give-up flag
    float *part_o = nullptr, *part_gu = nullptr, *part_dn = nullptr, *part_q = nullptr;   // one per GEMM of a launch
    void* xn2 = nullptr;                     // second packed operand (norm before the feed-forward block)
    float *ssq_a = nullptr, *ssq_f = nullptr;   // [d / 16][Mp] partial sums of squares of the two deferred norms
    unsigned* sync_ctr = nullptr;            // [(n_layers + 1)][FUSED_SYNC_WORDS] barrier counters, + the give-up flag
    unsigned* sync_abort = nullptr;
    unsigned long long sync_timeout_ticks = 5000000ull;     // 50 ms of the 100 MHz counter
    unsigned long long* timeline = nullptr;  // caller's buffer for the layer kernel's time stamps, or NULL
    size_t timeline_launches = 0;
    ScratchRows scratch;                     // as the last pass left it
    bool plan_missing = false;               // set by run_gemm if it ever had to skip a launch
    bool greedy_drafts = true;               // sd_greedy_step also runs the draft heads
    // float32 path (dtype SD_DTYPE_F32; f32.hip): weights [out][in] as float, natural activation layouts
    bool f32 = false;
    struct F32Layer { const float *attn_norm, *wqkv, *wo, *ffn_norm, *wgu, *wdown; };
    struct F32 {
        const float *embed, *lm_head, *final_norm, *medusa_w, *medusa_b;
        std::vector<F32Layer> layers;
        float *q, *attn, *act, *kt, *vt, *xh;
    } f;
};

// Handles get a process-wide serial number: graph keys use it instead of the handle's address, which a
// later handle can be given again after this one is destroyed.
static uint64_t next_uid() {
    static uint64_t n = 0;
    return ++n;
}

struct sd_kv {
    uint64_t uid = next_uid();
    const sd_model* m;
    int B, cap, cap_blocks;
    uint16_t* buf;
    size_t layer_stride;                     // elements between layers, per K or V plane
    uint16_t *kc, *vc;                       // plane bases
    float *kc32 = nullptr, *vc32 = nullptr;  // float32 models: planes [layer][seq][cap][d], layer_stride = B * cap * d
    int32_t* state = nullptr;                // device: kv_len, n_old, root_tok, last_row, cand, io scratch
    int32_t *kv_len, *n_old, *root_tok, *last_row, *cand, *i_nacc, *i_tokens, *i_slots;
    std::vector<int32_t> len_hi;             // host upper bound of the committed lengths
    bool has_draft = false;
};

struct sd_tree {
    uint64_t uid = next_uid();
    int T, Tp, H, topk;
    int32_t* dev = nullptr;                  // parent | depth | rank
    const int32_t *parent, *depth, *rank;
};

// ------------------------------------------------------------------------------------------ model
static int check_config(const sd_config* c) {
    if (c->dtype != SD_DTYPE_BF16 && c->dtype != SD_DTYPE_F32) return fail(SD_ERR_SHAPE, "dtype must be SD_DTYPE_BF16 or SD_DTYPE_F32");
    if (c->head_dim != 64 && c->head_dim != 128) return fail(SD_ERR_SHAPE, "head_dim must be 64 or 128");
    if (c->n_layers < 1 || c->n_heads < 1 || c->vocab < 2 || c->vocab > 163840) return fail(SD_ERR_SHAPE, "bad sizes");
    if (c->d_model != c->n_heads * c->head_dim) return fail(SD_ERR_SHAPE, "d_model != n_heads * head_dim");
    if (c->d_model % 32 || c->d_model > 8192) return fail(SD_ERR_SHAPE, "d_model must be a multiple of 32, <= 8192");
    if (c->d_ffn % 16 || c->d_ffn < 16) return fail(SD_ERR_SHAPE, "d_ffn must be a multiple of 16");
    if (c->n_medusa < 1 || c->n_medusa > SD_MAX_MEDUSA) return fail(SD_ERR_SHAPE, "n_medusa must be in 1..15");
    if (c->topk < 1 || c->topk > 32 || c->topk > c->vocab) return fail(SD_ERR_SHAPE, "topk must be in 1..32");
    if (c->trunc_fallback != SD_TRUNC_KEEP_ALL && c->trunc_fallback != SD_TRUNC_KEEP_ONE)
        return fail(SD_ERR_SHAPE, "bad trunc_fallback");
    if (!(c->rope_theta > 0.f) || !(c->rms_eps >= 0.f)) return fail(SD_ERR_SHAPE, "bad rope_theta / rms_eps");
    return SD_OK;
}

// The float32 model: weights copied as they are ([out][in] float; gate and up stacked, the draft heads stacked, a
// zero bias where none is given) and a workspace in natural row-major layouts. No launch plans, no packing.
static int create_f32(const sd_config* cfg, const sd_weights* w, int max_rows, hipStream_t s, sd_model** out) {
    const int L = cfg->n_layers, d = cfg->d_model, F = cfg->d_ffn, V = cfg->vocab, H = cfg->n_medusa, hd = cfg->head_dim;
    sd_model* m = new (std::nothrow) sd_model();
    if (!m) return fail(SD_ERR_HIP, "out of host memory");
    m->cfg = *cfg;
    m->f32 = true;
    m->max_rows = max_rows;
    m->MBmax = pow2_blocks(max_rows);
    m->Vpad = ceil_div(V, 32) * 32;
    const int Mp = m->MBmax * 32;
    const int HBp = pow2_blocks(H * SD_MAX_BATCH > 256 ? 256 : H * SD_MAX_BATCH) * 32;
    size_t sz = 0;
    auto take = [&](size_t floats) { size_t o = sz; sz = align_up(sz + floats * 4, 256); return o; };
    const size_t o_embed = take((size_t)V * d), o_lm = take((size_t)V * d), o_fn = take(d);
    const size_t o_mw = take((size_t)H * d * d), o_mb = take((size_t)H * d);
    std::vector<size_t> o_an(L), o_qkv(L), o_o(L), o_ffn(L), o_gu(L), o_dn(L);
    for (int l = 0; l < L; ++l) {
        o_an[l] = take(d); o_qkv[l] = take((size_t)3 * d * d); o_o[l] = take((size_t)d * d);
        o_ffn[l] = take(d); o_gu[l] = take((size_t)2 * F * d); o_dn[l] = take((size_t)d * F);
    }
    hipError_t e = hipMalloc((void**)&m->arena, sz);
    if (e != hipSuccess) { delete m; return fail(SD_ERR_HIP, "hipMalloc(%zu) for weights: %s", sz, hipGetErrorString(e)); }
    char* A = m->arena;
    auto copy = [&](size_t off, const void* src, size_t floats) {
        if (e == hipSuccess) e = hipMemcpyAsync(A + off, src, floats * 4, hipMemcpyDeviceToDevice, s);
        return (const float*)(A + off);
    };
    e = hipMemsetAsync(A + o_mb, 0, (size_t)H * d * 4, s);
    m->f.embed = copy(o_embed, w->embed, (size_t)V * d);
    m->f.lm_head = copy(o_lm, w->lm_head, (size_t)V * d);
    m->f.final_norm = copy(o_fn, w->final_norm, d);
    for (int i = 0; i < H; ++i) {
        copy(o_mw + (size_t)i * d * d * 4, w->medusa_w[i], (size_t)d * d);
        if (w->medusa_b && w->medusa_b[i]) copy(o_mb + (size_t)i * d * 4, w->medusa_b[i], d);
    }
    m->f.medusa_w = (const float*)(A + o_mw);
    m->f.medusa_b = (const float*)(A + o_mb);
    m->f.layers.resize(L);
    for (int l = 0; l < L; ++l) {
        sd_model::F32Layer& lw = m->f.layers[l];
        lw.attn_norm = copy(o_an[l], w->attn_norm[l], d);
        lw.wqkv = copy(o_qkv[l], w->wqkv[l], (size_t)3 * d * d);
        lw.wo = copy(o_o[l], w->wo[l], (size_t)d * d);
        lw.ffn_norm = copy(o_ffn[l], w->ffn_norm[l], d);
        lw.wgu = copy(o_gu[l], w->w_gate[l], (size_t)F * d);
        copy(o_gu[l] + (size_t)F * d * 4, w->w_up[l], (size_t)F * d);
        lw.wdown = copy(o_dn[l], w->w_down[l], (size_t)d * F);
    }
    m->embed = m->f.embed;

    size_t wz = 0;
    auto wtake = [&](size_t bytes) { size_t o = wz; wz = align_up(wz + bytes, 256); return o; };
    const size_t w_x = wtake((size_t)Mp * d * 4);
    const size_t w_logits = wtake((size_t)std::max(Mp, SD_MAX_BATCH) * m->Vpad * 4);
    const size_t w_hlog = wtake((size_t)HBp * m->Vpad * 4);
    const size_t w_q = wtake((size_t)Mp * d * 4), w_attn = wtake((size_t)Mp * d * 4), w_act = wtake((size_t)Mp * F * 4);
    const size_t w_kt = wtake((size_t)L * Mp * d * 4), w_vt = wtake((size_t)L * Mp * d * 4);
    const size_t w_xh = wtake((size_t)HBp * d * 4);
    const size_t w_tok = wtake((size_t)Mp * 4), w_pos = wtake((size_t)Mp * 4), w_anc = wtake((size_t)Mp * SD_ANC_WORDS * 4);
    const size_t w_cs = wtake((size_t)Mp * (hd / 2) * 8), w_g = wtake(3 * 4), w_fin = wtake(SD_MAX_BATCH * 4);
    const size_t w_best = wtake((size_t)std::max(Mp, SD_MAX_BATCH) * rank_chunks(V) * 8);
    const size_t w_rk = wtake((size_t)std::min(H * SD_MAX_BATCH, 256) * rank_chunks(V) * cfg->topk * 8);
    const size_t w_rm = wtake(sizeof(PassMap)), w_freq = wtake((size_t)(hd / 2) * 8);
    const size_t w_rs = wtake((size_t)Mp * 16), w_zs = wtake((size_t)ceil_div(V, 32) * 4);
    if (e == hipSuccess) e = hipMalloc((void**)&m->work, wz);
    if (e == hipSuccess) e = hipMemsetAsync(m->work, 0, wz, s);
    if (e != hipSuccess) {
        hipStreamSynchronize(s);
        hipFree(m->arena);
        if (m->work) hipFree(m->work);
        delete m;
        return fail(SD_ERR_HIP, "float32 model: weights or workspace: %s", hipGetErrorString(e));
    }
    char* Wk = m->work;
    m->x = (float*)(Wk + w_x); m->logits = (float*)(Wk + w_logits); m->hlogits = (float*)(Wk + w_hlog);
    m->f.q = (float*)(Wk + w_q); m->f.attn = (float*)(Wk + w_attn); m->f.act = (float*)(Wk + w_act);
    m->f.kt = (float*)(Wk + w_kt); m->f.vt = (float*)(Wk + w_vt); m->f.xh = (float*)(Wk + w_xh);
    m->rt.tok = (int32_t*)(Wk + w_tok); m->rt.pos = (int32_t*)(Wk + w_pos); m->rt.anc = (uint32_t*)(Wk + w_anc);
    m->rt.cs = (float2*)(Wk + w_cs);
    m->best = (float2*)(Wk + w_best); m->ranked = Wk + w_rk; m->fin_rows = (int32_t*)(Wk + w_fin);
    m->rm_dev = (PassMap*)(Wk + w_rm);
    m->row_stats = (float4*)(Wk + w_rs);
    m->g_parent = (int32_t*)(Wk + w_g); m->g_depth = m->g_parent + 1; m->g_rank = m->g_parent + 2;
    m->zero_stop = (uint32_t*)(Wk + w_zs);
    m->rope_freq = (double*)(Wk + w_freq);
    launch_rope_freqs(m->rope_freq, hd, cfg->rope_theta, s);
    launch_fill_i32(m->g_parent, -1, 1, s);
    e = hipStreamSynchronize(s);
    if (e == hipSuccess) e = hipGetLastError();
    if (e != hipSuccess) {
        hipFree(m->arena); hipFree(m->work); delete m;
        return fail(SD_ERR_HIP, "float32 model: set-up failed: %s", hipGetErrorString(e));
    }
    *out = m;
    return SD_OK;
}

extern "C" int sd_model_create(const sd_config* cfg, const sd_weights* w, int32_t max_rows, void* stream,
                               sd_model** out) {
    if (!cfg || !w || !out) return fail(SD_ERR_NULL, "sd_model_create: NULL argument");
    *out = nullptr;
    int rc = check_config(cfg);
    if (rc) return rc;
    if (max_rows < 1 || max_rows > 256) return fail(SD_ERR_SHAPE, "max_rows must be in 1..256");
    if (!w->embed || !w->lm_head || !w->final_norm || !w->attn_norm || !w->wqkv || !w->wo || !w->ffn_norm ||
        !w->w_gate || !w->w_up || !w->w_down || !w->medusa_w)
        return fail(SD_ERR_NULL, "sd_model_create: NULL weight pointer");
    const int L = cfg->n_layers, d = cfg->d_model, F = cfg->d_ffn, V = cfg->vocab, H = cfg->n_medusa;
    for (int l = 0; l < L; ++l)
        if (!w->attn_norm[l] || !w->wqkv[l] || !w->wo[l] || !w->ffn_norm[l] || !w->w_gate[l] || !w->w_up[l] ||
            !w->w_down[l])
            return fail(SD_ERR_NULL, "sd_model_create: NULL weight pointer in layer %d", l);
    for (int i = 0; i < H; ++i)
        if (!w->medusa_w[i]) return fail(SD_ERR_NULL, "sd_model_create: NULL draft-head weight %d", i);

    hipStream_t s = (hipStream_t)stream;
    if (cfg->dtype == SD_DTYPE_F32) return create_f32(cfg, w, max_rows, s, out);
    sd_model* m = new (std::nothrow) sd_model();
    if (!m) return fail(SD_ERR_HIP, "out of host memory");
    m->cfg = *cfg;
    m->max_rows = max_rows;
    m->MBmax = pow2_blocks(max_rows);
    m->KBd = d / 16;
    m->KBf = F / 16;
    m->Fpad = (int)align_up(F, 32);
    m->NBqkv = 3 * d / 32;
    m->NBo = d / 32;
    m->NBgu = 2 * m->Fpad / 32;
    m->NBv = ceil_div(V, 32);
    m->Vpad = m->NBv * 32;
    m->NBmed = H * d / 32;

    // ---- arena of packed weights
    const size_t frag = 1024;    // bytes per fragment
    size_t sz = 0;
    auto take = [&](size_t bytes) { size_t o = sz; sz = align_up(sz + bytes, 256); return o; };
    size_t o_embed = take((size_t)V * d * 2), o_lm = take((size_t)m->NBv * m->KBd * frag), o_fn = take((size_t)d * 2);
    size_t o_med = take((size_t)m->NBmed * m->KBd * frag);
    std::vector<size_t> o_mb(H), o_an(L), o_qkv(L), o_o(L), o_ffn(L), o_gu(L), o_dn(L);
    for (int i = 0; i < H; ++i) o_mb[i] = take((size_t)d * 2);
    for (int l = 0; l < L; ++l) {
        o_an[l] = take((size_t)d * 2);
        o_qkv[l] = take((size_t)m->NBqkv * m->KBd * frag);
        o_o[l] = take((size_t)m->NBo * m->KBd * frag);
        o_ffn[l] = take((size_t)d * 2);
        o_gu[l] = take((size_t)m->NBgu * m->KBd * frag);
        o_dn[l] = take((size_t)m->NBo * m->KBf * frag);
    }
    hipError_t e = hipMalloc((void**)&m->arena, sz);
    if (e != hipSuccess) { delete m; return fail(SD_ERR_HIP, "hipMalloc(%zu) for weights: %s", sz, hipGetErrorString(e)); }
    char* A = m->arena;
    auto copy = [&](size_t off, const void* src, size_t bytes) {
        return hipMemcpyAsync(A + off, src, bytes, hipMemcpyDeviceToDevice, s);
    };
    e = copy(o_embed, w->embed, (size_t)V * d * 2);
    if (e == hipSuccess) e = copy(o_fn, w->final_norm, (size_t)d * 2);
    if (e != hipSuccess) { hipFree(m->arena); delete m; return fail(SD_ERR_HIP, "weight copy: %s", hipGetErrorString(e)); }
    m->embed = A + o_embed;
    m->final_norm = A + o_fn;
    launch_pack_weight(w->lm_head, A + o_lm, V, d, 0, m->NBv, m->KBd, s);
    m->lm_head = A + o_lm;
    for (int i = 0; i < H; ++i) {
        launch_pack_weight(w->medusa_w[i], A + o_med, d, d, i * (d / 32), m->NBmed, m->KBd, s);
        if (w->medusa_b && w->medusa_b[i]) {
            if (e == hipSuccess) e = copy(o_mb[i], w->medusa_b[i], (size_t)d * 2);
            m->medusa_b.p[i] = (const uint16_t*)(A + o_mb[i]);
        } else {
            m->medusa_b.p[i] = nullptr;
        }
    }
    m->medusa_w = A + o_med;
    m->layers.resize(L);
    for (int l = 0; l < L; ++l) {
        LayerW& lw = m->layers[l];
        if (e == hipSuccess) e = copy(o_an[l], w->attn_norm[l], (size_t)d * 2);
        if (e == hipSuccess) e = copy(o_ffn[l], w->ffn_norm[l], (size_t)d * 2);
        launch_pack_weight(w->wqkv[l], A + o_qkv[l], 3 * d, d, 0, m->NBqkv, m->KBd, s);
        launch_pack_weight(w->wo[l], A + o_o[l], d, d, 0, m->NBo, m->KBd, s);
        launch_pack_weight(w->w_gate[l], A + o_gu[l], F, d, 0, m->NBgu, m->KBd, s);
        launch_pack_weight(w->w_up[l], A + o_gu[l], F, d, m->Fpad / 32, m->NBgu, m->KBd, s);
        launch_pack_weight(w->w_down[l], A + o_dn[l], d, F, 0, m->NBo, m->KBf, s);
        lw.attn_norm = A + o_an[l];
        lw.ffn_norm = A + o_ffn[l];
        lw.wqkv = A + o_qkv[l];
        lw.wo = A + o_o[l];
        lw.wgu = A + o_gu[l];
        lw.wdown = A + o_dn[l];
    }

    // ---- workspace
    const int Mp = m->MBmax * 32, nh = cfg->n_heads, hd = cfg->head_dim;
    const int ld_max = std::max(std::max(3 * d, 2 * m->Fpad), H * d);
    // launch plans for every GEMM shape this model can issue
    size_t pf = 0;
    std::vector<int32_t> cnt_all;
    std::vector<size_t> cnt_off;
    {
        const int shapes[6][2] = {{m->KBd, m->NBqkv}, {m->KBd, m->NBo}, {m->KBd, m->NBgu},
                                  {m->KBf, m->NBo},   {m->KBd, m->NBv}, {m->KBd, m->NBmed}};
        for (int mb = 1; mb <= 8; mb *= 2)
            for (int si = 0; si < 6; ++si) {
                const int* sh = shapes[si];
                // beyond MBmax only the LM head is used (draft-head rows); the draft-head
                // projection has one row block, or the step's when the heads run on every tree row
                if (mb > m->MBmax && si != 4) continue;
                bool dup = false;
                for (const GemmPlan& q : m->plans) dup |= q.MB == mb && q.KB == sh[0] && q.NB == sh[1];
                if (dup) continue;
                GemmPlan pl;
                std::vector<int32_t> cnt((sh[1] + 7) / 8 + 1, 0), slot0(256, 0);
                gemm_plan_make(&pl, mb, sh[0], sh[1], cnt.data(), slot0.data());
                cnt_off.push_back(cnt_all.size());
                cnt_all.insert(cnt_all.end(), cnt.begin(), cnt.end());
                cnt_all.insert(cnt_all.end(), slot0.begin(), slot0.end());
                m->plans.push_back(pl);
                pf = std::max(pf, (size_t)pl.slots_max * (mb * 32) * (size_t)sh[1] * 32);
            }
    }
    (void)ld_max;
    m->part_floats = pf;
    for (int r = 0; r < 2; ++r) {
        const int shapes[3][2] = {{m->KBd, m->NBqkv}, {m->KBd, m->NBo}, {m->KBf, m->NBo}};
        for (int i = 0; i < 3; ++i) {
            const int rows = 16 << r, KB = shapes[i][0], NB = shapes[i][1];
            m->kw[r][i] = (uint64_t)KB * NB < (1ull << 22) ? kw_plan(rows, KB, NB) : KwPlan{0, 0, 0};
            pf = std::max(pf, (size_t)m->kw[r][i].S * rows * (size_t)NB * 32);
        }
    }
    // Prompts: passes of up to 1024 rows (a model of max_rows > 128 has the room for prompt passes of 256). The time of a layer
    // of a pass decides how a prompt is cut (prompt_runs).
    size_t pf_prompt = pf;
    m->prompt_rows = m->MBmax == 8 ? PROMPT_ROWS : max_rows;
    if (m->MBmax == 8) {
        const int shapes[4][2] = {{m->KBd, m->NBqkv}, {m->KBd, m->NBo}, {m->KBd, m->NBgu}, {m->KBf, m->NBo}};
        m->prompt_us.assign(PROMPT_ROWS / 32 + 1, 0.0);
        for (int mb = 1; mb <= PROMPT_ROWS / 32; ++mb) {
            m->prompt_us[mb] = prompt_pass_us(shapes, mb * 32);
            if (mb <= 8) continue;
            for (int i = 0; i < 4; ++i) {
                GemmPlan pl;
                double cycles = 0;
                gemm_plan_prompt(&pl, mb, shapes[i][0], shapes[i][1], &cycles, i == 2);
                m->prompt_plans.push_back(pl);
                pf_prompt = std::max(pf_prompt, (size_t)pl.slots_max * mb * 32 * (size_t)shapes[i][1] * 32);
            }
        }
    }
    // rows of the buffers that a pass fills: packed rows, and rows padded to whole chunks (attention's side)
    const int Mr = std::max(m->MBmax * 32, m->MBmax == 8 ? PROMPT_ROWS : 0), Mc = std::max(m->MBmax * 32, m->MBmax == 8 ? PROMPT_PADDED : 0);
    m->max_parts = 65;
    const int HBp = pow2_blocks(std::min((H + 1) * SD_MAX_BATCH, 256)) * 32;      // head rows of a batch, and its base rows
    size_t wz = 0;
    auto wtake = [&](size_t bytes) { size_t o = wz; wz = align_up(wz + bytes, 256); return o; };
    size_t w_x = wtake((size_t)Mr * d * 4), w_part = wtake(pf_prompt * 4), w_logits = wtake((size_t)Mp * m->Vpad * 4);
    size_t w_hlog = wtake((size_t)HBp * m->Vpad * 4), w_hf = wtake((size_t)Mp * d * 4);
    size_t w_hrows = wtake((size_t)SD_MAX_BATCH * d * 4);
    size_t w_opart = wtake((size_t)Mp * nh * m->max_parts * hd * 4), w_ml = wtake((size_t)Mp * nh * m->max_parts * 8);
    size_t w_xn = wtake((size_t)std::max(Mr, HBp) * d * 4), w_attn = wtake((size_t)Mr * d * 4);
    size_t w_act = wtake((size_t)Mr * F * 4), w_q = wtake((size_t)Mc * d * 4);
    size_t w_kt = wtake((size_t)L * Mp * d * 2), w_vt = wtake((size_t)L * Mp * d * 2);
    size_t w_ktp = wtake(Mc > Mp ? (size_t)Mc * d * 2 : 0), w_vtp = wtake(Mc > Mp ? (size_t)Mc * d * 2 : 0);
    size_t w_tok = wtake((size_t)Mr * 4), w_pos = wtake((size_t)Mr * 4), w_anc = wtake((size_t)Mc * SD_ANC_WORDS * 4);
    size_t w_cs = wtake((size_t)Mr * (hd / 2) * 8), w_g = wtake(3 * 4), w_fin = wtake(SD_MAX_BATCH * 4);
    size_t w_best = wtake((size_t)std::max(Mp, SD_MAX_BATCH) * rank_chunks(V) * 8);
    size_t w_rk = wtake((size_t)std::min(H * SD_MAX_BATCH, 256) * rank_chunks(V) * cfg->topk * 8);
    size_t w_rs = wtake((size_t)Mp * 16), w_rm = wtake(sizeof(PassMap)), w_freq = wtake((size_t)(hd / 2) * 8);
    size_t w_xh = wtake(align_up((size_t)H * Mp, 256) * d * 4);
    size_t w_zs = wtake((size_t)ceil_div(V, 32) * 4), w_zf = wtake(2048);
    size_t w_ssqa = wtake((size_t)align_up(d / 16, 4) * Mp * 4), w_ssqf = wtake((size_t)align_up(d / 16, 4) * Mp * 4);
    size_t w_xn2 = wtake((size_t)Mp * d * 4);
    // the persistent layer kernel: partial sums of each of its four GEMMs in a buffer of their own, a second
    // packed operand, and the barrier counters of every launch of a pass
    int dev_now = 0;
    const bool fused_fits = hipGetDevice(&dev_now) == hipSuccess && fused_max_resident(dev_now) >= 256;
    size_t w_po = 0, w_pgu = 0, w_pdn = 0, w_pq = 0, w_sync = 0;
    if (fused_fits) {
        w_po = wtake(pf * 4); w_pgu = wtake(pf * 4); w_pdn = wtake(pf * 4); w_pq = wtake(pf * 4);
        w_sync = wtake(((size_t)(L + 1) * FUSED_SYNC_WORDS + 64) * 4);
    }
    if (e != hipSuccess) {                             // one of the per-layer / per-head weight copies was refused
        hipStreamSynchronize(s);
        hipFree(m->arena); delete m;
        return fail(SD_ERR_HIP, "weight copy: %s", hipGetErrorString(e));
    }
    e = hipMalloc((void**)&m->work, wz);
    if (e == hipSuccess) e = hipMalloc((void**)&m->plan_cnt, cnt_all.size() * 4);
    if (e == hipSuccess) e = hipMemcpy(m->plan_cnt, cnt_all.data(), cnt_all.size() * 4, hipMemcpyHostToDevice);
    if (e != hipSuccess) {
        hipFree(m->arena);
        if (m->work) hipFree(m->work);
        if (m->plan_cnt) hipFree(m->plan_cnt);
        delete m;
        return fail(SD_ERR_HIP, "hipMalloc(%zu) for workspace: %s", wz, hipGetErrorString(e));
    }
    for (size_t i = 0; i < m->plans.size(); ++i) {
        m->plans[i].cnt_dev = m->plan_cnt + cnt_off[i];
        m->plans[i].slot0_dev = m->plans[i].cnt_dev + (m->plans[i].NB + 7) / 8 + 1;      // right behind the counts
    }
    e = hipMemsetAsync(m->work, 0, wz, s);
    if (e != hipSuccess) {
        hipStreamSynchronize(s);
        hipFree(m->arena); hipFree(m->work); hipFree(m->plan_cnt); delete m;
        return fail(SD_ERR_HIP, "workspace clear: %s", hipGetErrorString(e));
    }
    char* Wk = m->work;
    m->x = (float*)(Wk + w_x); m->part = (float*)(Wk + w_part); m->logits = (float*)(Wk + w_logits);
    m->hlogits = (float*)(Wk + w_hlog); m->hf = (float*)(Wk + w_hf); m->h_rows = (float*)(Wk + w_hrows);
    m->opart = (float*)(Wk + w_opart); m->mlpart = (float2*)(Wk + w_ml);
    m->xn = Wk + w_xn; m->attn_x = Wk + w_attn; m->act = Wk + w_act; m->q = Wk + w_q;
    m->kt = Wk + w_kt; m->vt = Wk + w_vt;
    m->ktp = Wk + w_ktp; m->vtp = Wk + w_vtp;
    m->xh = Wk + w_xh;
    m->rt.tok = (int32_t*)(Wk + w_tok); m->rt.pos = (int32_t*)(Wk + w_pos); m->rt.anc = (uint32_t*)(Wk + w_anc);
    m->rt.cs = (float2*)(Wk + w_cs);
    m->best = (float2*)(Wk + w_best); m->ranked = Wk + w_rk; m->fin_rows = (int32_t*)(Wk + w_fin);
    m->rm_dev = (PassMap*)(Wk + w_rm);
    m->row_stats = (float4*)(Wk + w_rs);
    m->g_parent = (int32_t*)(Wk + w_g); m->g_depth = m->g_parent + 1; m->g_rank = m->g_parent + 2;
    m->zero_stop = (uint32_t*)(Wk + w_zs);
    m->zfrag = Wk + w_zf;
    m->ssq_a = (float*)(Wk + w_ssqa); m->ssq_f = (float*)(Wk + w_ssqf);
    m->xn2 = Wk + w_xn2;
    if (fused_fits) {
        m->part_o = (float*)(Wk + w_po); m->part_gu = (float*)(Wk + w_pgu); m->part_dn = (float*)(Wk + w_pdn);
        m->part_q = (float*)(Wk + w_pq);
        m->sync_ctr = (unsigned*)(Wk + w_sync);
        m->sync_abort = m->sync_ctr + (size_t)(L + 1) * FUSED_SYNC_WORDS;
        m->fused_ok = true;
    }
    m->rope_freq = (double*)(Wk + w_freq);
    launch_rope_freqs(m->rope_freq, hd, cfg->rope_theta, s);
    launch_fill_i32(m->g_parent, -1, 1, s);
    e = hipStreamSynchronize(s);
    if (e == hipSuccess) e = hipGetLastError();
    if (e != hipSuccess) {
        hipFree(m->arena); hipFree(m->work); hipFree(m->plan_cnt); delete m;
        return fail(SD_ERR_HIP, "weight packing failed: %s", hipGetErrorString(e));
    }
    *out = m;
    return SD_OK;
}

static void prof_free(sd_model* m) {
    for (hipEvent_t e : m->prof.ev) hipEventDestroy(e);
    m->prof = Profile();
}

extern "C" int sd_profile_begin(sd_model* m, int32_t max_launches) {
    if (!m) return fail(SD_ERR_NULL, "sd_profile_begin: NULL model");
    if (max_launches < 1 || max_launches > (1 << 20)) return fail(SD_ERR_SHAPE, "sd_profile_begin: bad max_launches");
    prof_free(m);
    m->prof.ev.resize((size_t)max_launches * 2);
    m->prof.cls.assign(max_launches, 0);
    m->prof.bytes.assign(max_launches, 0.0);
    for (size_t i = 0; i < m->prof.ev.size(); ++i) {
        hipError_t e = hipEventCreate(&m->prof.ev[i]);
        if (e != hipSuccess) {
            m->prof.ev.resize(i);
            prof_free(m);
            return fail(SD_ERR_HIP, "hipEventCreate: %s", hipGetErrorString(e));
        }
    }
    m->prof.on = true;
    return SD_OK;
}

extern "C" int sd_profile_end(sd_model* m, void* stream, double* ms_total, int64_t* launches, double* bytes_total) {
    if (!m || !ms_total || !launches || !bytes_total) return fail(SD_ERR_NULL, "sd_profile_end: NULL argument");
    if (!m->prof.on) return fail(SD_ERR_STATE, "sd_profile_end: profiling is not on");
    hipError_t e = hipStreamSynchronize((hipStream_t)stream);
    if (e != hipSuccess) { prof_free(m); return fail(SD_ERR_HIP, "sync: %s", hipGetErrorString(e)); }
    for (int c = 0; c < PROF_CLASSES; ++c) { ms_total[c] = 0.0; launches[c] = 0; bytes_total[c] = 0.0; }
    for (size_t i = 0; i < m->prof.used; ++i) {
        float ms = 0.f;
        e = hipEventElapsedTime(&ms, m->prof.ev[2 * i], m->prof.ev[2 * i + 1]);
        if (e != hipSuccess) { prof_free(m); return fail(SD_ERR_HIP, "hipEventElapsedTime: %s", hipGetErrorString(e)); }
        int c = m->prof.cls[i];
        ms_total[c] += ms;
        launches[c] += 1;
        bytes_total[c] += m->prof.bytes[i];
    }
    prof_free(m);
    return SD_OK;
}

extern "C" int sd_build_labels(const int32_t* l0, int32_t batch, int32_t seq, int32_t n_heads, int32_t frag_id,
                               int32_t pad_id, int32_t ignore_id, int32_t no_frag, int32_t* labels, void* stream) {
    if (batch < 1 || batch > 65535 || seq < 0) return fail(SD_ERR_SHAPE, "sd_build_labels: bad batch or seq");
    if (n_heads < 0 || n_heads > SD_LABELS_MAX_HEADS)
        return fail(SD_ERR_SHAPE, "sd_build_labels: n_heads must be in 0..%d", SD_LABELS_MAX_HEADS);
    if (no_frag != SD_LABELS_KEEP_BASE && no_frag != SD_LABELS_KEEP_ALL)
        return fail(SD_ERR_SHAPE, "sd_build_labels: bad no_frag policy");
    if (seq == 0) return SD_OK;                        // nothing to write; the pointers are not looked at
    if (!l0 || !labels) return fail(SD_ERR_NULL, "sd_build_labels: NULL argument");
    launch_build_labels(l0, batch, seq, n_heads, frag_id, pad_id, ignore_id, no_frag == SD_LABELS_KEEP_ALL, labels,
                        (hipStream_t)stream);
    HIP_TRY(hipGetLastError());
    return SD_OK;
}

extern "C" int sd_set_draft_schedule(sd_model* m, int32_t schedule) {
    if (!m) return fail(SD_ERR_NULL, "sd_set_draft_schedule: NULL model");
    if (schedule != SD_DRAFT_AFTER_ACCEPT && schedule != SD_DRAFT_ALL_NODES)
        return fail(SD_ERR_SHAPE, "sd_set_draft_schedule: unknown schedule %d", schedule);
    m->draft_schedule = schedule;
    return SD_OK;
}

extern "C" int sd_set_fused(sd_model* m, int32_t on) {
    if (!m) return fail(SD_ERR_NULL, "sd_set_fused: NULL model");
    m->use_fused = on != 0;
    return SD_OK;
}

extern "C" int sd_set_layer_timeline(sd_model* m, void* dev_buf, size_t bytes) {
    if (!m) return fail(SD_ERR_NULL, "sd_set_layer_timeline: NULL model");
    if (dev_buf && (((uintptr_t)dev_buf) & 7)) return fail(SD_ERR_SHAPE, "sd_set_layer_timeline: buffer must be 8-byte aligned");
    m->timeline = (unsigned long long*)dev_buf;
    m->timeline_launches = dev_buf ? bytes / ((size_t)24 * 256 * 8) : 0;
    return SD_OK;
}

extern "C" int sd_set_sync_timeout(sd_model* m, int64_t microseconds) {
    if (!m) return fail(SD_ERR_NULL, "sd_set_sync_timeout: NULL model");
    if (microseconds < 0 || microseconds > 10000000) return fail(SD_ERR_SHAPE, "sd_set_sync_timeout: 0 .. 10 s");
    m->sync_timeout_ticks = (unsigned long long)microseconds * 100ull;
    return SD_OK;
}

// Has a workgroup of the persistent kernel given up a wait since the last look? Called where the host has just
// synchronised the stream anyway. The flag is cleared, so one failure is reported once.
static int check_fused_abort(sd_model* m, const char* who) {
    if (!m->fused_dirty || !m->sync_abort) return SD_OK;
    unsigned flag = 0;
    HIP_TRY(hipMemcpy(&flag, m->sync_abort, 4, hipMemcpyDeviceToHost));
    m->fused_dirty = false;
    if (flag) {
        HIP_TRY(hipMemset(m->sync_abort, 0, 4));
        return fail(SD_ERR_HIP, "%s: a wait between workgroups inside the layer kernel ran out of time; the results "
                    "enqueued since the last successful check are invalid", who);
    }
    return SD_OK;
}

extern "C" int sd_set_greedy_drafts(sd_model* m, int32_t on) {
    if (!m) return fail(SD_ERR_NULL, "sd_set_greedy_drafts: NULL model");
    m->greedy_drafts = on != 0;
    return SD_OK;
}

extern "C" int sd_set_graph_mode(sd_model* m, int32_t on) {
    if (!m) return fail(SD_ERR_NULL, "sd_set_graph_mode: NULL model");
    m->use_graphs = on != 0;
    return SD_OK;
}

extern "C" int sd_model_destroy(sd_model* m) {
    if (!m) return SD_OK;
    for (sd_model::StepGraph& g : m->graphs) hipGraphExecDestroy(g.exec);
    m->graphs.clear();
    if (m->cap_stream) { hipStreamDestroy(m->cap_stream); m->cap_stream = nullptr; }
    prof_free(m);
    hipFree(m->arena);
    hipFree(m->work);
    hipFree(m->plan_cnt);
    delete m;
    return SD_OK;
}

// ------------------------------------------------------------------------------------------ KV cache
extern "C" size_t sd_kv_bytes(const sd_config* cfg, int32_t batch, int32_t cap) {
    if (!cfg || batch < 1 || cap < 1) return 0;
    if (cfg->dtype == SD_DTYPE_F32)
        return (size_t)cfg->n_layers * 2 * batch * cap * cfg->n_heads * cfg->head_dim * 4;
    size_t blocks = (size_t)ceil_div(cap, 32);
    return (size_t)cfg->n_layers * 2 * batch * cfg->n_heads * blocks * 32 * cfg->head_dim * 2;
}

extern "C" int sd_kv_create(const sd_model* m, int32_t batch, int32_t cap, void* dev_buf, size_t bytes, sd_kv** out) {
    if (!m || !dev_buf || !out) return fail(SD_ERR_NULL, "sd_kv_create: NULL argument");
    *out = nullptr;
    if (batch < 1 || batch > SD_MAX_BATCH) return fail(SD_ERR_SHAPE, "batch must be in 1..%d", SD_MAX_BATCH);
    if (batch * m->cfg.n_medusa > 256) return fail(SD_ERR_SHAPE, "batch * n_medusa must be <= 256");
    if (cap < m->cfg.n_medusa + 2) return fail(SD_ERR_SHAPE, "cap too small");
    if (bytes < sd_kv_bytes(&m->cfg, batch, cap)) return fail(SD_ERR_SHAPE, "KV buffer too small");
    if (((uintptr_t)dev_buf) & 15) return fail(SD_ERR_SHAPE, "KV buffer must be 16-byte aligned");
    sd_kv* kv = new (std::nothrow) sd_kv();
    if (!kv) return fail(SD_ERR_HIP, "out of host memory");
    kv->m = m;
    kv->B = batch;
    kv->cap = cap;
    kv->cap_blocks = ceil_div(cap, 32);
    kv->buf = (uint16_t*)dev_buf;
    kv->layer_stride = (size_t)batch * m->cfg.n_heads * kv->cap_blocks * 32 * m->cfg.head_dim;
    kv->kc = kv->buf;
    kv->vc = kv->buf + (size_t)m->cfg.n_layers * kv->layer_stride;
    if (m->f32) {
        kv->layer_stride = (size_t)batch * cap * m->cfg.d_model;
        kv->kc32 = (float*)dev_buf;
        kv->vc32 = kv->kc32 + (size_t)m->cfg.n_layers * kv->layer_stride;
    }
    const int H = m->cfg.n_medusa, k = m->cfg.topk;
    const int W = std::max(H + 1, SD_MAX_TREE);
    size_t n = (size_t)batch * (4 + H * k + 1 + 2 * W);
    hipError_t e = hipMalloc((void**)&kv->state, n * 4);
    if (e != hipSuccess) { delete kv; return fail(SD_ERR_HIP, "hipMalloc state: %s", hipGetErrorString(e)); }
    e = hipMemset(kv->state, 0, n * 4);
    // The cache itself starts as zeros: attention multiplies the value rows of a partly filled block by
    // probabilities that are exactly 0 for the rows past the committed length, and 0 * NaN is NaN, so no
    // row the kernels can touch may hold a non-finite bit pattern left behind by the buffer's last user.
    if (e == hipSuccess) e = hipMemset(dev_buf, 0, sd_kv_bytes(&m->cfg, batch, cap));
    if (e == hipSuccess) e = hipDeviceSynchronize();
    if (e != hipSuccess) { hipFree(kv->state); delete kv; return fail(SD_ERR_HIP, "hipMemset: %s", hipGetErrorString(e)); }
    int32_t* p = kv->state;
    kv->kv_len = p; p += batch;
    kv->n_old = p; p += batch;
    kv->root_tok = p; p += batch;
    kv->last_row = p; p += batch;
    kv->cand = p; p += (size_t)batch * H * k;
    kv->i_nacc = p; p += batch;
    kv->i_tokens = p; p += (size_t)batch * W;
    kv->i_slots = p;
    kv->len_hi.assign(batch, 0);
    *out = kv;
    return SD_OK;
}

extern "C" int sd_kv_destroy(sd_kv* kv) {
    if (!kv) return SD_OK;
    hipFree(kv->state);
    delete kv;
    return SD_OK;
}

extern "C" int sd_kv_len(sd_kv* kv, int32_t* out_len, void* stream) {
    if (!kv || !out_len) return fail(SD_ERR_NULL, "sd_kv_len: NULL argument");
    HIP_TRY(hipMemcpyAsync(out_len, kv->kv_len, kv->B * 4, hipMemcpyDeviceToHost, (hipStream_t)stream));
    HIP_TRY(hipStreamSynchronize((hipStream_t)stream));
    for (int b = 0; b < kv->B; ++b) kv->len_hi[b] = out_len[b];
    if (int rc = check_fused_abort(const_cast<sd_model*>(kv->m), "sd_kv_len")) return rc;
    return SD_OK;
}

extern "C" int sd_kv_set_len(sd_kv* kv, const int32_t* len, void* stream) {
    if (!kv || !len) return fail(SD_ERR_NULL, "sd_kv_set_len: NULL argument");
    for (int b = 0; b < kv->B; ++b)
        if (len[b] < 0 || len[b] > kv->cap) return fail(SD_ERR_SHAPE, "sd_kv_set_len: length %d out of range", len[b]);
    // a replay would set the device's lengths behind the host's bounds on them
    hipStreamCaptureStatus cap = hipStreamCaptureStatusNone;
    HIP_TRY(hipStreamIsCapturing((hipStream_t)stream, &cap));
    if (cap != hipStreamCaptureStatusNone) return fail(SD_ERR_STATE, "sd_kv_set_len: the stream is being captured");
    launch_set_i32(len, kv->kv_len, kv->B, (hipStream_t)stream);
    HIP_TRY(hipGetLastError());
    for (int b = 0; b < kv->B; ++b) kv->len_hi[b] = len[b];
    return SD_OK;
}

static int kv_rows_common(sd_kv* kv, int layer, int seq, int row0, int nrows, void* k_rows, void* v_rows, int to_cache,
                          void* stream) {
    if (!kv || !k_rows || !v_rows) return fail(SD_ERR_NULL, "sd_kv_*_rows: NULL argument");
    const sd_config& c = kv->m->cfg;
    if (layer < 0 || layer >= c.n_layers || seq < 0 || seq >= kv->B || row0 < 0 || nrows < 0 || row0 + nrows > kv->cap)
        return fail(SD_ERR_SHAPE, "sd_kv_*_rows: index out of range");
    if (nrows == 0) return SD_OK;
    if (kv->m->f32) {
        const size_t o = layer * kv->layer_stride + (size_t)seq * kv->cap * c.d_model;
        launch_f32_kv_rows(kv->kc32 + o, kv->vc32 + o, (float*)k_rows, (float*)v_rows, row0, nrows, c.d_model, to_cache,
                           (hipStream_t)stream);
        HIP_TRY(hipGetLastError());
        return SD_OK;
    }
    size_t off = layer * kv->layer_stride + (size_t)seq * c.n_heads * kv->cap_blocks * 32 * c.head_dim;
    launch_kv_rows(kv->kc + off, kv->vc + off, k_rows, v_rows, row0, nrows, c.n_heads, c.head_dim, kv->cap_blocks,
                   to_cache, (hipStream_t)stream);
    HIP_TRY(hipGetLastError());
    return SD_OK;
}
extern "C" int sd_kv_write_rows(sd_kv* kv, int32_t layer, int32_t seq, int32_t row0, int32_t nrows, const void* k_rows,
                                const void* v_rows, void* stream) {
    return kv_rows_common(kv, layer, seq, row0, nrows, (void*)k_rows, (void*)v_rows, 1, stream);
}
extern "C" int sd_kv_read_rows(sd_kv* kv, int32_t layer, int32_t seq, int32_t row0, int32_t nrows, void* k_rows,
                               void* v_rows, void* stream) {
    return kv_rows_common(kv, layer, seq, row0, nrows, k_rows, v_rows, 0, stream);
}

extern "C" int sd_kv_set_draft(sd_kv* kv, const int32_t* root_tok, const int32_t* cand, void* stream) {
    if (!kv || !root_tok || !cand) return fail(SD_ERR_NULL, "sd_kv_set_draft: NULL argument");
    const sd_config& c = kv->m->cfg;
    launch_copy_i32(root_tok, kv->root_tok, kv->B, cand, kv->cand, kv->B * c.n_medusa * c.topk, (hipStream_t)stream);
    HIP_TRY(hipGetLastError());
    kv->has_draft = true;
    return SD_OK;
}
extern "C" int sd_kv_get_draft(sd_kv* kv, int32_t* root_tok, int32_t* cand, void* stream) {
    if (!kv || !root_tok || !cand) return fail(SD_ERR_NULL, "sd_kv_get_draft: NULL argument");
    const sd_config& c = kv->m->cfg;
    launch_copy_i32(kv->root_tok, root_tok, kv->B, kv->cand, cand, kv->B * c.n_medusa * c.topk, (hipStream_t)stream);
    HIP_TRY(hipGetLastError());
    return SD_OK;
}

// ------------------------------------------------------------------------------------------ tree
static int validate_tree(int T, const int32_t* parent, const int32_t* depth, const int32_t* rank, int H, int k) {
    if (T < 1 || T > SD_MAX_TREE) return fail(SD_ERR_BAD_TREE, "tree must have 1..%d nodes", SD_MAX_TREE);
    if (parent[0] != -1 || depth[0] != 0) return fail(SD_ERR_BAD_TREE, "node 0 must be the root (parent -1, depth 0)");
    for (int j = 1; j < T; ++j) {
        if (parent[j] < 0 || parent[j] >= j) return fail(SD_ERR_BAD_TREE, "node %d: parent must precede it", j);
        if (depth[j] != depth[parent[j]] + 1) return fail(SD_ERR_BAD_TREE, "node %d: depth != parent's depth + 1", j);
        if (depth[j] > H) return fail(SD_ERR_BAD_TREE, "node %d: depth %d exceeds the number of draft heads", j, depth[j]);
        if (rank[j] < 0 || rank[j] >= k) return fail(SD_ERR_BAD_TREE, "node %d: rank out of range", j);
        for (int i = 1; i < j; ++i)
            if (parent[i] == parent[j] && rank[i] == rank[j])
                return fail(SD_ERR_BAD_TREE, "nodes %d and %d: siblings with equal rank", i, j);
    }
    return SD_OK;
}

extern "C" int sd_tree_create(int32_t T, const int32_t* parent, const int32_t* depth, const int32_t* rank,
                              int32_t n_medusa, int32_t topk, sd_tree** out) {
    if (!parent || !depth || !rank || !out) return fail(SD_ERR_NULL, "sd_tree_create: NULL argument");
    *out = nullptr;
    if (n_medusa < 0 || n_medusa > SD_MAX_MEDUSA || topk < 1) return fail(SD_ERR_SHAPE, "bad n_medusa / topk");
    int rc = validate_tree(T, parent, depth, rank, n_medusa, topk);
    if (rc) return rc;
    sd_tree* t = new (std::nothrow) sd_tree();
    if (!t) return fail(SD_ERR_HIP, "out of host memory");
    t->T = T;
    t->Tp = ceil_div(T, 32) * 32;
    t->H = n_medusa;
    t->topk = topk;
    hipError_t e = hipMalloc((void**)&t->dev, (size_t)3 * T * 4);
    if (e == hipSuccess) e = hipMemcpy(t->dev, parent, (size_t)T * 4, hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemcpy(t->dev + T, depth, (size_t)T * 4, hipMemcpyHostToDevice);
    if (e == hipSuccess) e = hipMemcpy(t->dev + 2 * T, rank, (size_t)T * 4, hipMemcpyHostToDevice);
    if (e != hipSuccess) {
        if (t->dev) hipFree(t->dev);
        delete t;
        return fail(SD_ERR_HIP, "tree upload: %s", hipGetErrorString(e));
    }
    t->parent = t->dev;
    t->depth = t->dev + T;
    t->rank = t->dev + 2 * T;
    *out = t;
    return SD_OK;
}

extern "C" int sd_tree_destroy(sd_tree* t) {
    if (!t) return SD_OK;
    hipFree(t->dev);
    delete t;
    return SD_OK;
}

// ------------------------------------------------------------------------------------------ forward
// Layers 0..L-1 on the rows described by m->rt / m->x (B sequences of Tp rows each). Leaves the
// last down-projection's partial sums in m->part (added by the caller's next norm).
// Claims the next pair of profile events (or -1): the launcher hands them to the kernel launch, which
// stamps them with the kernel's own start and end, so launch gaps are not counted.
static int prof_claim(sd_model* m, int cls, double bytes) {
    Profile& p = m->prof;
    if (!p.on || p.used * 2 + 1 >= p.ev.size()) return -1;
    int i = (int)p.used++;
    p.cls[i] = cls;
    p.bytes[i] = bytes;
    return i;
}
static hipEvent_t prof_ev(sd_model* m, int i, int which) { return i >= 0 ? m->prof.ev[2 * i + which] : nullptr; }

// One weight-streaming GEMM; algorithmic bytes = one read of the (unpadded) weight matrix.
static SkRowScale row_scale(const sd_model* m, const float* ssq) {
    return SkRowScale{ssq, m->cfg.d_model / 16, 1.f / (float)m->cfg.d_model, m->cfg.rms_eps};
}
static const SkRowScale NO_SCALE = {nullptr, 0, 0.f, 0.f};

static PartView run_gemm(sd_model* m, const void* Xp, const void* Wp, float* out, int rows, int MB, int KB, int NB, int n_real,
                         hipStream_t s, void* swiglu = nullptr) {
    const GemmPlan* p = m->find_plan(MB, KB, NB);
    if (!p) {                                          // unreachable after have_plans(); never launch with another shape's plan
        m->plan_missing = true;
        return PartView{out, 0, NB * 32, nullptr, 0};  // no slots: the consumer adds nothing
    }
    const int pi = prof_claim(m, PROF_GEMM, (double)n_real * KB * 16 * 2);
    return launch_gemm(*p, Xp, Wp, m->zfrag, out, rows, s, prof_ev(m, pi, 0), prof_ev(m, pi, 1), swiglu, m->KBf);
}

// ---- a handful of rows (few.hip): no packed operands, no partial sums
// Do M rows against a packed matrix of KB x NB fragments go that way?
static bool few_rows(int M, int KB, int NB) { return M <= FEW_ROWS && (uint64_t)KB * NB < (1ull << 22); }
static FewLinear few_linear(const float* X, int ldx, const void* W, int KB, int NB, int M, int units, float* out, int ldo) {
    FewLinear a;
    memset(&a, 0, sizeof(a));
    a.X = X; a.ldx = ldx; a.W = (const bf16x8*)W; a.KB = KB; a.NB = NB; a.M = M; a.n_units = units; a.out = out; a.ldo = ldo;
    return a;
}
static FewLinear few_norm_linear(const sd_model* m, const void* gain, const int32_t* gather, const void* W, int NB, int M, int units,
                                 float* out, int ldo) {
    FewLinear a = few_linear(m->x, m->cfg.d_model, W, m->KBd, NB, M, units, out, ldo);
    a.gain = (const uint16_t*)gain; a.eps = m->cfg.rms_eps; a.gather = gather;
    return a;
}
template <class F>
static void few_launch(sd_model* m, int n_real, int KB, F&& launch) {
    const int pi = prof_claim(m, PROF_GEMM, (double)n_real * KB * 16 * 2);
    launch(prof_ev(m, pi, 0), prof_ev(m, pi, 1));
}
// LM head of `rows` rows of X (through the final norm, or as they are): dense logits
static PartView few_lm_head(sd_model* m, const float* X, const float* row_scale, bool norm, int rows, hipStream_t s) {
    FewLinear a = norm ? few_norm_linear(m, m->final_norm, nullptr, m->lm_head, m->NBv, rows, m->NBv * 2, m->part, m->Vpad)
                       : few_linear(X, m->cfg.d_model, m->lm_head, m->KBd, m->NBv, rows, m->NBv * 2, m->part, m->Vpad);
    a.row_scale = row_scale;
    few_launch(m, m->cfg.vocab, m->KBd, [&](hipEvent_t e0, hipEvent_t e1) { launch_few_store(a, s, e0, e1); });
    return PartView{m->part, 0, m->Vpad, nullptr, 1};
}
// Draft heads (and with base the rows themselves in front) at rows gather[b] of the residual stream, and the LM head of all
// of those rows: the partial sums of its logits.
static PartView few_drafts(sd_model* m, const int32_t* gather, int base, int n, hipStream_t s) {
    const int H = m->cfg.n_medusa, d = m->cfg.d_model, rows = n * (H + base), MB = pow2_blocks(rows);
    const bool wide = !few_rows(rows, m->KBd, m->NBv);
    FewLinear a = few_norm_linear(m, m->final_norm, gather, m->medusa_w, m->NBmed, n, m->NBmed * 2, (float*)m->xn, d);
    a.base = base;
    a.scale_out = m->h_rows;
    if (wide) { a.packed = (bf16x8*)m->xn; a.MB = MB; }
    few_launch(m, H * d, m->KBd, [&](hipEvent_t e0, hipEvent_t e1) { launch_few_heads(a, m->medusa_b, s, e0, e1); });
    if (wide) return run_gemm(m, m->xn, m->lm_head, m->part, rows, MB, m->KBd, m->NBv, m->cfg.vocab, s);
    return few_lm_head(m, (const float*)m->xn, m->h_rows, false, rows, s);
}
static bool few_layers(const sd_model* m, int M) {
    return M <= FEW_LAYER_ROWS && few_rows(M, m->KBd, m->NBgu) && few_rows(M, m->KBd, m->NBqkv) && few_rows(M, m->KBf, m->NBo);
}

// Every GEMM shape a pass over M rows issues (and, with heads = true, the draft heads after it, in the
// schedule given) has a launch plan: checked by the entry points before anything is enqueued.
static bool have_plans(const sd_model* m, int M, int B, bool heads, bool all_rows) {
    if (m->f32) return true;                           // the float32 kernels take any shape
    const int MB = pow2_blocks(M), H = m->cfg.n_medusa;
    bool ok = m->find_plan(MB, m->KBd, m->NBqkv) && m->find_plan(MB, m->KBd, m->NBo) && m->find_plan(MB, m->KBd, m->NBgu) &&
              m->find_plan(MB, m->KBf, m->NBo) && m->find_plan(MB, m->KBd, m->NBv);
    if (heads && !all_rows)
        ok = ok && m->find_plan(1, m->KBd, m->NBmed) && m->find_plan(pow2_blocks(H * B), m->KBd, m->NBv);
    if (heads && all_rows) {
        const int R = H * M, n_chunks = ceil_div(R, 256);
        ok = ok && m->find_plan(MB, m->KBd, m->NBmed) && m->find_plan(pow2_blocks(R - (n_chunks - 1) * 256), m->KBd, m->NBv) &&
             (n_chunks == 1 || m->find_plan(8, m->KBd, m->NBv));
    }
    return ok;
}

// Does a pass over M rows run through the persistent layer kernel?
static bool fused_eligible(const sd_model* m, int M) {
    if (m->f32) return false;
    const int MB = pow2_blocks(M);
    return m->use_fused && m->fused_ok && (MB == 1 || MB == 2 || MB == 8);
}
// The geometry that the pass over B sequences of Tp rows will launch: worked out once per pass, launched, and part of the
// key under which the pass is captured. (float32 attention has no parts: none of its launches depends on n_hi.)
struct PassGeom : AttnGeom { AttnSplit split; int whole; };     // whole: 0, or the parts of attn_whole.hip (1: none)
// M: the pass's rows (a short prompt has fewer than its padded B * Tp).
static PassGeom pass_geometry(const sd_model* m, const sd_kv* kv, const int32_t* seq, int B, int M, int Tp, int n_hi) {
    PassGeom g = {};
    if (m->f32) return g;
    // (a batch is cut sequence by sequence once its longest one has 256 rows)
    static_cast<AttnGeom&>(g) = attn_geometry_of_pass(fused_eligible(m, B * Tp), m->cfg.n_heads, m->max_parts, B, Tp, n_hi,
                                                      B > 1 && n_hi >= 256);
    // (a handful of rows take the merged parts as an operand of another layout)
    g.whole = !fused_eligible(m, B * Tp) && !few_layers(m, M) ? attn_whole_parts(m->cfg.n_heads, B, Tp, n_hi) : 0;
    if (g.whole > 1) g.nparts = g.whole;
    if (g.per == 0) {
        int len[SD_MAX_BATCH];
        for (int i = 0; i < B; ++i) len[i] = kv->len_hi[seq ? seq[i] : i];
        g.split = attn_split(m->cfg.n_heads, B, len);
        g.ncparts = g.nparts = g.split.max_parts;
    }
    return g;
}

// A projection of a pass of M rows: k_gemm_kw where the pass has a plan for it (kw: or NULL), else the split over column groups.
static PartView run_projection(sd_model* m, const KwPlan* kw, const void* X, const void* W, int M, int MB, int KB, int NB, int n_real,
                               hipStream_t s) {
    if (!kw || !kw->C) return run_gemm(m, X, W, m->part, M, MB, KB, NB, n_real, s);
    KwLinear a;
    memset(&a, 0, sizeof(a));
    a.X = X; a.W = W; a.KB = KB; a.NB = NB; a.M = M; a.S = kw->S; a.n_units = NB * 2; a.out = m->part; a.ldo = NB * 32;
    a.slot_stride = (size_t)kw->RT * 16 * a.ldo;
    few_launch(m, n_real, KB, [&](hipEvent_t e0, hipEvent_t e1) { launch_gemm_kw(*kw, a, s, e0, e1); });
    return PartView{m->part, a.slot_stride, a.ldo, nullptr, kw->S};
}

static PartView run_layers(sd_model* m, sd_kv* kv, RowRef rr, const RowMap& rm, int B, int M, int Tp, int n_hi, const PassGeom& ag,
                           hipStream_t s) {
    const sd_config& c = m->cfg;
    const int MB = pow2_blocks(M), d = c.d_model, nh = c.n_heads, hd = c.head_dim, TB = Tp / 32;
    PartView prev = {nullptr, 0, d, nullptr, 0};
    const size_t t_stride = (size_t)B * nh * TB * 32 * hd;     // elements per layer of tree scratch
    const int longest = *std::max_element(rm.len, rm.len + B);
    const bool few = few_layers(m, M);
    const KwPlan* kw = M <= 32 ? m->kw[M <= 16 ? 0 : 1] : nullptr;
    const auto plan = [&](int which) { return kw ? kw + which : nullptr; };
    for (int l = 0; l < c.n_layers; ++l) {
        const LayerW& lw = m->layers[l];
        PartView pq = {m->part, 0, 3 * d, nullptr, 1};
        if (few) {
            const FewLinear a = few_norm_linear(m, lw.attn_norm, nullptr, lw.wqkv, m->NBqkv, M, 3 * d / 16, m->part, 3 * d);
            few_launch(m, 3 * d, m->KBd, [&](hipEvent_t e0, hipEvent_t e1) { launch_few_store(a, s, e0, e1); });
        } else {
            launch_norm_pack(m->x, prev, lw.attn_norm, c.rms_eps, m->xn, nullptr, M, d, MB, nullptr, s);
            pq = run_projection(m, plan(KW_QKV), m->xn, lw.wqkv, M, MB, m->KBd, m->NBqkv, 3 * d, s);
        }
        uint16_t* kt = (uint16_t*)m->kt + l * t_stride;
        uint16_t* vt = (uint16_t*)m->vt + l * t_stride;
        // With one query group per head (trees of up to 64 nodes, plain decoding, short prompt chunks) the attention
        // launch builds the queries and the tree's keys / values from the QKV partial sums itself: one launch less per
        // layer (7B shape: plain decoding +3 %, the 64-node step 4.95 -> 4.89 ms once each of its two tree blocks has a
        // workgroup of its own to build it). With several query groups every group would repeat that work, and at long
        // contexts, where the tree blocks go to the last of several cache parts, that part would become the straggler
        // (16 k rows: attention 55 -> 64 us): there the stage stays a launch of its own. Where every (sequence, head) has
        // ONE workgroup (a batch that fills the chip) all workgroups carry the same extra work, none is a straggler, and
        // the launch saved is worth more than it costs (batch of eight 32-node trees: attention 65.4 -> 72.8 us, the
        // 11.8 us launch gone, step -0.8 %); so it is with the parts of a batch that is cut sequence by sequence, the last of
        // which takes the tree.
        const AttnSplit* split = ag.split.n ? &ag.split : nullptr;
        const bool fr = Tp <= 64 && (ag.whole || ag.tree_sep || ag.ncparts == 1 || split);
        if (!fr) launch_rope_kv(pq, m->rt, rr, m->q, kt, vt, B, Tp, nh, hd, s);
        // algorithmic bytes: one read of K and V of the committed rows (upper bound n_hi) + tree rows
        const int pa = prof_claim(m, PROF_ATTN, (double)B * (n_hi + Tp) * 2.0 * d * 2.0);
        const uint16_t *kc = kv->kc + l * kv->layer_stride, *vc = kv->vc + l * kv->layer_stride;
        if (ag.whole)
            launch_attn_whole(m->q, kc, vc, kt, vt, kv->kv_len, m->rt.anc, m->attn_x, rr, B, nh, hd, Tp, kv->cap_blocks, MB, s,
                              prof_ev(m, pa, 0), prof_ev(m, pa, 1), fr ? &pq : nullptr, fr ? &m->rt : nullptr, ag.whole, m->opart, m->mlpart);
        else
            launch_tree_attn(m->q, kc, vc, kt, vt, kv->kv_len, m->rt.anc, m->opart, m->mlpart, rr, B, nh, hd, Tp, kv->cap_blocks,
                             ag.ncparts, ag.per, ag.tree_sep, s, prof_ev(m, pa, 0), prof_ev(m, pa, 1), fr ? &pq : nullptr,
                             fr ? &m->rt : nullptr, split);
        if (few) {
            FewLinear a = few_linear(nullptr, 0, lw.wo, m->KBd, m->NBo, M, d / 16, m->x, d);
            a.Xp = (const bf16x8*)m->attn_x;
            if (rr.map == nullptr && few_merges(M, d)) {      // the projection merges the attention parts itself
                a.opart = m->opart; a.mlpart = m->mlpart; a.nh = nh; a.hd = hd; a.Tp = Tp; a.nparts = ag.nparts; a.R = rr.R;
                for (int& own : a.own) own = ag.nparts;
                for (int i = 0; i < ag.split.n; ++i) a.own[ag.split.slot[i] & 255] = ag.split.slot[i] >> 16;
            } else {
                launch_attn_merge_few(m->opart, m->mlpart, m->attn_x, rr, longest, B, nh, hd, Tp, ag.nparts, s, split);
            }
            few_launch(m, d, m->KBd, [&](hipEvent_t e0, hipEvent_t e1) { launch_few_add(a, s, e0, e1); });
            a = few_norm_linear(m, lw.ffn_norm, nullptr, lw.wgu, m->NBgu, M, c.d_ffn / 16, nullptr, 0);
            a.up = m->Fpad / 16;
            a.packed = (bf16x8*)m->act;
            few_launch(m, 2 * c.d_ffn, m->KBd, [&](hipEvent_t e0, hipEvent_t e1) { launch_few_swiglu(a, s, e0, e1); });
            a = few_linear(nullptr, 0, lw.wdown, m->KBf, m->NBo, M, d / 16, m->x, d);
            a.Xp = (const bf16x8*)m->act;
            few_launch(m, d, m->KBf, [&](hipEvent_t e0, hipEvent_t e1) { launch_few_add(a, s, e0, e1); });
            continue;                                  // (prev stays empty: the residual stream is complete)
        }
        if (ag.whole != 1) launch_attn_merge(m->opart, m->mlpart, m->attn_x, rr, longest, B, nh, hd, Tp, ag.nparts, MB, s, split);
        PartView po = run_projection(m, plan(KW_O), m->attn_x, lw.wo, M, MB, m->KBd, m->NBo, d, s);
        launch_norm_pack(m->x, po, lw.ffn_norm, c.rms_eps, m->xn, nullptr, M, d, MB, nullptr, s);
        PartView pg = run_gemm(m, m->xn, lw.wgu, m->part, M, MB, m->KBd, m->NBgu, 2 * c.d_ffn, s);
        launch_swiglu_pack(pg, c.d_ffn, m->Fpad, m->act, M, MB, s);
        prev = run_projection(m, plan(KW_DOWN), m->act, lw.wdown, M, MB, m->KBf, m->NBo, d, s);
    }
    return prev;
}

// ---- the same pass through the persistent layer kernel: one launch per layer besides attention
static FusedGemm fused_gemm(const sd_model* m, int MB, int KB, int NB, const void* X, const void* W, float* out) {
    const GemmPlan* p = m->find_plan(MB, KB, NB);          // present: have_plans() ran before
    FusedGemm g;
    g.X = (const bf16x8*)X; g.W = (const bf16x8*)W; g.out = out;
    g.KB = KB; g.NB = NB; g.ldo = NB * 32;
    g.slot_stride = (size_t)MB * 32 * g.ldo;
    g.upw = p->upw; g.rem = p->rem; g.G = p->G; g.nmax = p->slots;
    g.kb_magic = (uint32_t)((0x100000000ull + (uint64_t)KB - 1) / (uint64_t)KB);
    g.slot0 = p->slot0_dev;
    g.cnt = p->uniform ? nullptr : p->cnt_dev;
    g.sc = NO_SCALE;
    return g;
}
// Layers 0..L-1 and, with want_lm, the final norm and the LM-head GEMM, whose partial sums the returned view
// describes (without want_lm: the last down projection's, still to be added to m->x).
// (Its phases take the rows as [sequence][Tp]: the row map says off[i] = i * Tp.)
static PartView run_forward_fused(sd_model* m, sd_kv* kv, RowRef rr, int B, int Tp, int n_hi, const PassGeom& ag, bool want_lm,
                                  hipStream_t s) {
    const sd_config& c = m->cfg;
    const int M = B * Tp, MB = pow2_blocks(M), d = c.d_model, nh = c.n_heads, hd = c.head_dim, TB = Tp / 32, L = c.n_layers;
    const size_t t_stride = (size_t)B * nh * TB * 32 * hd;
    launch_fill_i32((int32_t*)m->sync_ctr, 0, (L + 1) * FUSED_SYNC_WORDS, s);
    m->fused_dirty = true;
    FusedArgs a;
    memset(&a, 0, sizeof(a));
    a.M = M; a.MB = MB; a.B = B; a.Tp = Tp; a.d = d; a.nh = nh; a.hd = hd; a.F = c.d_ffn; a.Fpad = m->Fpad;
    a.nparts = ag.nparts; a.eps = c.rms_eps;
    a.x = m->x; a.opart = m->opart; a.mlpart = m->mlpart; a.att = (bf16x8*)m->attn_x;
    a.xn_f = (bf16x8*)m->xn2; a.act = (bf16x8*)m->act; a.xn_a = (bf16x8*)m->xn;
    a.ssq_f = m->ssq_f; a.ssq_a = m->ssq_a;
    a.rt = m->rt; a.q = (bf16x8*)m->q; a.zfrag = (const bf16x8*)m->zfrag;
    a.sync.abort_flag = m->sync_abort; a.sync.timeout_ticks = m->sync_timeout_ticks;
    const double w_attn_side = (double)(3 * d) * m->KBd * 32.0, w_ffn_side = ((double)d * m->KBd + 2.0 * c.d_ffn * m->KBd + (double)d * m->KBf) * 32.0;
    PartView last = {nullptr, 0, d, nullptr, 0};
    for (int l = 0; l <= L; ++l) {                         // launch l: the end of layer l-1 and the start of layer l
        double bytes = 0.0;
        a.phases = 0;
        a.sync.counters = m->sync_ctr + (size_t)l * FUSED_SYNC_WORDS;
        if (l > 0) {
            const LayerW& lw = m->layers[l - 1];
            a.phases |= FUSED_GEMM_O | FUSED_GEMM_GU | FUSED_GEMM_DN;
            a.g_o = fused_gemm(m, MB, m->KBd, m->NBo, m->attn_x, lw.wo, m->part_o);
            a.gain_f = (const uint16_t*)lw.ffn_norm;
            a.g_gu = fused_gemm(m, MB, m->KBd, m->NBgu, m->xn2, lw.wgu, m->part_gu);
            a.g_gu.sc = row_scale(m, m->ssq_f);
            a.g_dn = fused_gemm(m, MB, m->KBf, m->NBo, m->act, lw.wdown, m->part_dn);
            bytes += w_ffn_side;
            last = PartView{a.g_dn.out, a.g_dn.slot_stride, a.g_dn.ldo, a.g_dn.cnt, a.g_dn.nmax};
        }
        a.prev = PartView{nullptr, 0, d, nullptr, 0};
        if (l < L) {
            const LayerW& lw = m->layers[l];
            a.phases |= FUSED_GEMM_Q | FUSED_ROPE;
            a.gain_a = (const uint16_t*)lw.attn_norm;
            a.g_q = fused_gemm(m, MB, m->KBd, m->NBqkv, m->xn, lw.wqkv, m->part_q);
            a.g_q.sc = row_scale(m, m->ssq_a);
            a.kt = (uint16_t*)m->kt + l * t_stride;
            a.vt = (uint16_t*)m->vt + l * t_stride;
            bytes += w_attn_side;
        } else if (want_lm) {
            a.phases |= FUSED_GEMM_Q;
            a.gain_a = (const uint16_t*)m->final_norm;
            a.g_q = fused_gemm(m, MB, m->KBd, m->NBv, m->xn, m->lm_head, m->part_q);
            a.g_q.sc = row_scale(m, m->ssq_a);
            bytes += (double)c.vocab * m->KBd * 32.0;
            last = PartView{a.g_q.out, a.g_q.slot_stride, a.g_q.ldo, a.g_q.cnt, a.g_q.nmax};
        }
        a.timeline = (m->timeline && (size_t)l < m->timeline_launches) ? m->timeline + (size_t)l * 24 * 256 : nullptr;
        const int pi = prof_claim(m, PROF_GEMM, bytes);
        launch_layer(a, 256, s, prof_ev(m, pi, 0), prof_ev(m, pi, 1));
        if (l < L) {
            const int pa = prof_claim(m, PROF_ATTN, (double)B * (n_hi + Tp) * 2.0 * d * 2.0);
            launch_tree_attn(m->q, kv->kc + l * kv->layer_stride, kv->vc + l * kv->layer_stride, a.kt, a.vt, kv->kv_len,
                             m->rt.anc, m->opart, m->mlpart, rr, B, nh, hd, Tp, kv->cap_blocks, ag.ncparts, ag.per, ag.tree_sep, s,
                             prof_ev(m, pa, 0), prof_ev(m, pa, 1));
        }
    }
    return last;
}

// ------------------------------------------------------------------------------------------ float32 pass
// by_seq: slots, counts and old lengths are listed by sequence of the cache (else by sequence of the pass)
static void commit_rows(sd_model* m, sd_kv* kv, const ScratchRows& sc, bool by_seq, const int32_t* slots, const int32_t* n_acc,
                        int W, hipStream_t s) {
    const sd_config& c = m->cfg;
    // Entry of the lists and last row in one word: read from another line of the arguments, the last row costs the bfloat16
    // kernel 0.2 us of a step's 6.6.
    static_assert(SD_MAX_BATCH <= 256, "an entry fits 8 bits");
    RowMap rm;
    memset(&rm, 0, sizeof(rm));
    for (int i = 0; i < sc.n; ++i) { rm.seq[i] = sc.seq[i]; rm.off[i] = (by_seq ? sc.seq[i] : i) + 256 * (sc.len[i] - 1); }
    if (m->f32)
        launch_f32_kv_commit(m->f.kt, m->f.vt, kv->kc32, kv->vc32, slots, n_acc, kv->n_old, rm, sc.row0, kv->B, c.n_layers, sc.n,
                             c.d_model, sc.M, kv->cap, W, s);
    else
        launch_kv_commit(m->kt, m->vt, kv->kc, kv->vc, slots, n_acc, kv->n_old, rm, kv->B, c.n_layers, sc.n, c.n_heads,
                         c.head_dim, sc.Tp / 32, kv->cap_blocks, W, s);
}

static void run_forward_f32(sd_model* m, sd_kv* kv, RowRef rr, const RowMap& rm, int B, int M, int Tp, bool want_lm,
                            hipStream_t s) {
    const sd_config& c = m->cfg;
    const int d = c.d_model, F = c.d_ffn, longest = *std::max_element(rm.len, rm.len + B);
    sd_model::F32& f = m->f;
    for (int l = 0; l < c.n_layers; ++l) {
        const sd_model::F32Layer& lw = f.layers[l];
        float* kt = f.kt + (size_t)l * M * d;
        float* vt = f.vt + (size_t)l * M * d;
        launch_f32_qkv(m->x, lw.attn_norm, c.rms_eps, lw.wqkv, m->rt, f.q, kt, vt, M, c.n_heads, c.head_dim, s);
        launch_f32_attn(f.q, kv->kc32 + l * kv->layer_stride, kv->vc32 + l * kv->layer_stride, kt, vt, kv->kv_len, m->rt.anc,
                        f.attn, rr, longest, B, c.n_heads, c.head_dim, Tp, kv->cap, s);
        launch_f32_add_linear(f.attn, lw.wo, m->x, M, d, d, s);
        launch_f32_gate_up(m->x, lw.ffn_norm, c.rms_eps, lw.wgu, f.act, M, F, d, s);
        launch_f32_add_linear(f.act, lw.wdown, m->x, M, d, F, s);
    }
    if (want_lm)
        launch_f32_norm_linear(m->x, nullptr, f.final_norm, c.rms_eps, f.lm_head, m->logits, M, c.vocab, d, m->Vpad, s);
}
// dense float32 logits as the ranking kernels take them
static PartView dense_logits(const sd_model* m, const float* logits) { return PartView{logits, 0, m->Vpad, nullptr, 1}; }

static void run_draft_heads_f32(sd_model* m, sd_kv* kv, const int32_t* rows, int B, const SeqList& sl, float* head_logits_out,
                                hipStream_t s) {
    const sd_config& c = m->cfg;
    const int d = c.d_model, H = c.n_medusa;
    sd_model::F32& f = m->f;
    launch_f32_heads(m->x, rows, f.final_norm, c.rms_eps, f.medusa_w, f.medusa_b, f.xh, B, H, d, s);
    launch_f32_norm_linear(f.xh, nullptr, nullptr, 0.f, f.lm_head, m->hlogits, H * B, c.vocab, d, m->Vpad, s);
    launch_topk(dense_logits(m, m->hlogits), 0, c.vocab, c.topk, kv->cand, B, H, sl, head_logits_out, m->ranked, s);
}

// Final norm and LM head of all M rows: partial sums of the logits.
// (keep_h: also leaves the normalised rows in m->hf as fp32, for draft heads on every row)
static PartView run_lm_head(sd_model* m, PartView prev, int M, hipStream_t s, bool keep_h) {
    const sd_config& c = m->cfg;
    const int MB = pow2_blocks(M);
    if (!keep_h && prev.nmax == 0 && few_rows(M, m->KBd, m->NBv)) return few_lm_head(m, nullptr, nullptr, true, M, s);
    launch_norm_pack(m->x, prev, m->final_norm, c.rms_eps, m->xn, keep_h ? m->hf : nullptr, M, c.d_model, MB, nullptr, s);
    return run_gemm(m, m->xn, m->lm_head, m->part, M, MB, m->KBd, m->NBv, c.vocab, s);
}

// len: real rows of sequence i (NULL: T each)
static ScratchRows scratch_of_pass(const sd_kv* kv, const RowMap& rm, int n, int M, int Tp, const int32_t* len, int T) {
    ScratchRows sc;
    sc.B = kv->B; sc.Tp = Tp; sc.M = M; sc.n = n;
    for (int i = 0; i < n; ++i) { sc.seq[i] = rm.seq[i]; sc.row0.seq[i] = rm.off[i]; sc.len[i] = len ? len[i] : T; }
    return sc;
}

// The whole verifying pass: layers, and with want_lm the final norm and the LM head; returns the partial sums of the logits
// (without want_lm: of the last down projection, still to be added to m->x). Sequence i's rows start at row i * R (R = 0:
// at rm.off[i], prompt chunks).
static PartView run_forward(sd_model* m, sd_kv* kv, const RowMap& rm, int B, int M, int R, int Tp, int n_hi, const PassGeom& ag,
                            bool want_lm, bool keep_h, hipStream_t s) {
    const RowRef rr = {R ? nullptr : m->rm_dev, R};
    if (m->f32) { run_forward_f32(m, kv, rr, rm, B, M, Tp, want_lm, s); return dense_logits(m, m->logits); }
    if (fused_eligible(m, B * Tp)) {
        // (when the final norm's rows themselves are wanted, the last stage runs as kernels of its own)
        PartView pl = run_forward_fused(m, kv, rr, B, Tp, n_hi, ag, want_lm && !keep_h, s);
        return want_lm && keep_h ? run_lm_head(m, pl, M, s, true) : pl;
    }
    PartView prev = run_layers(m, kv, rr, rm, B, M, Tp, n_hi, ag, s);
    return want_lm ? run_lm_head(m, prev, M, s, keep_h) : prev;
}

static SeqList every_sequence() {
    SeqList sl;
    for (int b = 0; b < SD_MAX_BATCH; ++b) sl.seq[b] = b;
    return sl;
}

// draft heads at row last_row[b] of every sequence -> cand
static void run_draft_heads(sd_model* m, sd_kv* kv, int B, float* head_logits_out, hipStream_t s) {
    const sd_config& c = m->cfg;
    const int d = c.d_model, H = c.n_medusa;
    if (m->f32) { run_draft_heads_f32(m, kv, kv->last_row, B, every_sequence(), head_logits_out, s); return; }
    const PartView none = {nullptr, 0, d, nullptr, 0};
    if (few_rows(B, m->KBd, m->NBmed)) {
        const PartView pl = few_drafts(m, kv->last_row, 0, B, s);
        launch_topk(pl, 0, c.vocab, c.topk, kv->cand, B, H, every_sequence(), head_logits_out, m->ranked, s);
        return;
    }
    launch_norm_pack(m->x, none, m->final_norm, c.rms_eps, m->xn, m->h_rows, B, d, 1, kv->last_row, s);
    PartView pm = run_gemm(m, m->xn, m->medusa_w, m->part, B, 1, m->KBd, m->NBmed, H * d, s);
    const int MBh = pow2_blocks(H * B);
    launch_medusa_act(pm, m->h_rows, m->medusa_b, 0, B, H, d, m->xn, MBh * 32, MBh, MBh, s);
    PartView pl = run_gemm(m, m->xn, m->lm_head, m->part, H * B, MBh, m->KBd, m->NBv, c.vocab, s);
    launch_topk(pl, 0, c.vocab, c.topk, kv->cand, B, H, every_sequence(), head_logits_out, m->ranked, s);
}

// The end of a pass whose drafting rows are known before its logits are (plain decoding: every row; a prompt: the last
// row of the sequences that end, `gather`): final norm, base logits and draft heads of those n rows, with one pass of the
// LM head for the n base rows and the n * H head rows together. Leaves the base rows' ranking in m->best; logits: or NULL.
static void run_known_rows(sd_model* m, sd_kv* kv, PartView prev, int n, const int32_t* gather, const SeqList& sl, float* logits,
                           int ld, float* head_logits_out, hipStream_t s) {
    const sd_config& c = m->cfg;
    const int d = c.d_model, H = c.n_medusa;
    if (m->f32) {
        launch_f32_norm_linear(m->x, gather, m->f.final_norm, c.rms_eps, m->f.lm_head, m->logits, n, c.vocab, d, m->Vpad, s);
        launch_rank_best(dense_logits(m, m->logits), 0, n, c.vocab, logits, ld, m->best, s);
        run_draft_heads_f32(m, kv, gather, n, sl, head_logits_out, s);
        return;
    }
    if (prev.nmax == 0 && few_rows(n, m->KBd, m->NBmed) && n * (H + 1) <= 256) {
        const PartView pl = few_drafts(m, gather, 1, n, s);
        launch_rank_best(pl, 0, n, c.vocab, logits, ld, m->best, s);
        launch_topk(pl, n, c.vocab, c.topk, kv->cand, n, H, sl, head_logits_out, m->ranked, s);
        return;
    }
    launch_norm_pack(m->x, prev, m->final_norm, c.rms_eps, m->xn, m->h_rows, n, d, 1, gather, s);
    const int base = n * (H + 1) <= 256 ? 1 : 0;           // (the widest GEMM; beyond it two passes)
    if (!base) {
        PartView pb = run_gemm(m, m->xn, m->lm_head, m->part, n, 1, m->KBd, m->NBv, c.vocab, s);
        launch_rank_best(pb, 0, n, c.vocab, logits, ld, m->best, s);
    }
    PartView pm = run_gemm(m, m->xn, m->medusa_w, m->part, n, 1, m->KBd, m->NBmed, H * d, s);
    const int rows = n * (H + base), MBh = pow2_blocks(rows);
    launch_medusa_act(pm, m->h_rows, m->medusa_b, base, n, H, d, m->xn, MBh * 32, MBh, MBh, s);
    PartView pl = run_gemm(m, m->xn, m->lm_head, m->part, rows, MBh, m->KBd, m->NBv, c.vocab, s);
    if (base) launch_rank_best(pl, 0, n, c.vocab, logits, ld, m->best, s);
    launch_topk(pl, base * n, c.vocab, c.topk, kv->cand, n, H, sl, head_logits_out, m->ranked, s);
}

// The other schedule: the draft heads run on all M rows of the verifying pass (m->xn and m->hf
// still hold the final norm's output), the shared LM head on all H*M head rows in chunks of 256
// rows, and only the H rows of every sequence's last kept row (kv->last_row, set by the acceptance kernel) are
// summed out of the partial tiles and ranked.
static void run_draft_heads_all_rows(sd_model* m, sd_kv* kv, int B, int M, float* head_logits_out, hipStream_t s) {
    const sd_config& c = m->cfg;
    const int d = c.d_model, H = c.n_medusa, MB = pow2_blocks(M), R = H * M, CH = 256;
    PartView pm = run_gemm(m, m->xn, m->medusa_w, m->part, M, MB, m->KBd, m->NBmed, H * d, s);
    const int n_chunks = ceil_div(R, CH), MBlast = pow2_blocks(R - (n_chunks - 1) * CH);
    launch_medusa_act(pm, m->hf, m->medusa_b, 0, M, H, d, m->xh, CH, CH / 32, MBlast, s);
    for (int ch = 0; ch < n_chunks; ++ch) {
        const int rows = std::min(CH, R - ch * CH);
        const char* xc = (const char*)m->xh + (size_t)ch * CH * d * 4;
        PartView pl = run_gemm(m, xc, m->lm_head, m->part, rows, ch == n_chunks - 1 ? MBlast : CH / 32, m->KBd, m->NBv,
                               c.vocab, s);
        launch_reduce_selected(pl, m->hlogits, kv->last_row, B, H, M, ch * CH, rows, s);
    }
    launch_topk(dense_logits(m, m->hlogits), 0, c.vocab, c.topk, kv->cand, B, H, every_sequence(), head_logits_out, m->ranked, s);
}

// ------------------------------------------------------------------------------------------ prefill
// A prompt pass holds the next tokens of every sequence whose prompt has not ended, up to 256 rows in all and Tp per sequence
// (a prompt that has ended takes no rows).
struct PromptChunk { int b, tok, len, before; bool ends; };   // sequence, first token, tokens, rows earlier in the launch, ends its prompt
struct PromptPass { int Tp, M; std::vector<PromptChunk> chunks; };
static std::vector<PromptPass> cut_prompts(const sd_model* m, const int32_t* lens, int B) {
    std::vector<int> next(B), left(lens, lens + B);
    for (int b = 0, o = 0; b < B; ++b) { next[b] = o; o += lens[b]; }
    std::vector<PromptPass> passes;
    for (;;) {
        int A = 0;
        for (int b = 0; b < B; ++b) A += left[b] > 0;
        if (A == 0) return passes;
        PromptPass p;
        p.Tp = std::min(m->max_rows / A / 32 * 32, 256);       // (the widest GEMM of a pass on its own)
        p.M = 0;
        for (int b = 0; b < B; ++b) {
            if (left[b] <= 0) continue;
            const int n = std::min(left[b], p.Tp);
            p.chunks.push_back({b, next[b], n, 0, n == left[b]});
            next[b] += n;
            left[b] -= n;
            p.M += n;
        }
        passes.push_back(p);
    }
}

// The chunks of passes[0 .. n) as one launch sequence takes them: chunks of a sequence that follow one another joined up to
// 256 rows, those of passes[n - 1] left alone where a later commit is to find them (keep).
static std::vector<PromptChunk> joined_chunks(const PromptPass* passes, int n, bool keep, int* Tp) {
    std::vector<PromptChunk> v;
    int done[SD_MAX_BATCH] = {};                           // rows of the sequence so far
    *Tp = 0;
    for (int i = 0; i < n; ++i)
        for (const PromptChunk& c : passes[i].chunks) {
            PromptChunk* last = nullptr;                   // the sequence's latest
            for (PromptChunk& e : v)
                if (e.b == c.b) last = &e;
            if (last && !(keep && i == n - 1) && last->len + c.len <= 256) {
                last->len += c.len;
                last->ends = c.ends;
            } else {
                v.push_back(c);
                v.back().before = done[c.b];
            }
            done[c.b] += c.len;
        }
    for (const PromptChunk& c : v) *Tp = std::max(*Tp, ceil_div(c.len, 32) * 32);
    return v;
}

// Which passes run as one: as many as its buffers hold, where that is the sooner done.
static std::vector<int> join_passes(const sd_model* m, const std::vector<PromptPass>& passes) {
    const int n = (int)passes.size();
    if (m->prompt_rows <= 256 || fused_eligible(m, 256)) return std::vector<int>(n, 1);
    return prompt_runs(
        n,
        [&](int i, int k) {
            int M = 0, Tp;
            for (int j = i; j < i + k; ++j) M += passes[j].M;
            if (k == 1) return M;
            if (M > m->prompt_rows) return 0;
            const std::vector<PromptChunk> v = joined_chunks(&passes[i], k, i + k == n, &Tp);
            return v.size() > SD_MAX_BATCH || (int)v.size() * Tp > PROMPT_PADDED ? 0 : M;
        },
        [&](int rows) { return m->prompt_us[prompt_blocks(rows)]; });
}

// The sequences whose prompts end with these chunks: their last rows (of the pass), and themselves.
static int ending_rows(const std::vector<PromptChunk>& chunks, const RowMap& rm, SeqList* last, SeqList* fin) {
    int n = 0;
    for (size_t i = 0; i < chunks.size(); ++i)
        if (chunks[i].ends) {
            last->seq[n] = rm.off[i] + chunks[i].len - 1;
            fin->seq[n++] = chunks[i].b;
        }
    return n;
}

// What the ended prompts' sequences carry into their first step.
static void draft_from_prompts(sd_model* m, sd_kv* kv, PartView prev, int n_fin, const SeqList& fin, hipStream_t s) {
    if (!n_fin) return;
    run_known_rows(m, kv, prev, n_fin, m->fin_rows, fin, nullptr, 0, nullptr, s);
    launch_pick_root(m->best, m->cfg.vocab, kv->root_tok, n_fin, fin, s);
}

static void run_prompt_pass(sd_model* m, sd_kv* kv, const int32_t* tokens, const PromptPass& p, hipStream_t s) {
    const sd_config& c = m->cfg;
    const int A = (int)p.chunks.size(), Tp = p.Tp;
    ChainArgs ca;
    RowMap rm;
    SeqList fin, last;
    memset(&ca, 0, sizeof(ca));
    memset(&rm, 0, sizeof(rm));
    memset(&fin, 0, sizeof(fin));
    memset(&last, 0, sizeof(last));
    int M = 0, n_hi = 0;
    const bool padded = fused_eligible(m, A * Tp);         // that pass takes the rows as [sequence][Tp]
    for (int i = 0; i < A; ++i) {
        const PromptChunk& ch = p.chunks[i];
        ca.len[i] = ch.len;
        ca.off[i] = ch.tok;
        rm.seq[i] = ch.b;
        rm.off[i] = M;
        rm.len[i] = padded ? Tp : ch.len;
        M += rm.len[i];
        n_hi = std::max(n_hi, kv->len_hi[ch.b]);
    }
    const int n_fin = ending_rows(p.chunks, rm, &last, &fin);
    launch_build_rows_chain(m->rt, tokens, ca, rm, m->rm_dev, kv->kv_len, A, Tp, c.head_dim, m->rope_freq, m->embed, m->f32 ? 1 : 0,
                            c.d_model, c.vocab, m->x, s);
    const PassGeom ag = pass_geometry(m, kv, rm.seq, A, M, Tp, n_hi);
    PartView prev = run_forward(m, kv, rm, A, M, 0, Tp, n_hi, ag, false, false, s);
    launch_prefill_commit_setup(ca, rm, A, Tp, kv->i_slots, kv->i_nacc, kv->n_old, kv->kv_len, m->fin_rows, n_fin, last, s);
    m->scratch = scratch_of_pass(kv, rm, A, M, Tp, ca.len, 0);
    commit_rows(m, kv, m->scratch, false, kv->i_slots, kv->i_nacc, Tp, s);
    for (const PromptChunk& ch : p.chunks) kv->len_hi[ch.b] += ch.len;
    draft_from_prompts(m, kv, prev, n_fin, fin, s);
}

// Several passes (more than 256 rows) as one: every projection reads its weights once and has rows enough to fill the chip
// without cutting the contraction into partial sums. Attention takes the chunks as sequences of their own: a chunk attends
// the committed rows and its sequence's earlier chunks from the cache, where the rotary stage of the layer has put them, and
// its own rows from the pass's scratch. So the rows are committed layer by layer and nothing is left to commit at the end; what
// sd_kv_commit_rows may ask for afterwards, the rows of the last pass, goes to the model's scratch as if that pass had
// run by itself (last: it is the last of the call).
static void run_prompt_passes(sd_model* m, sd_kv* kv, const int32_t* tokens, const PromptPass* passes, int n, bool is_last,
                              hipStream_t s) {
    const sd_config& c = m->cfg;
    const int d = c.d_model, nh = c.n_heads, hd = c.head_dim;
    int Tp;
    const std::vector<PromptChunk> chunks = joined_chunks(passes, n, is_last, &Tp);
    const int V = (int)chunks.size(), keep = is_last ? V - (int)passes[n - 1].chunks.size() : V, keep_Tp = passes[n - 1].Tp;
    ChainArgs ca, sum;
    RowMap rm, seqs;
    SeqList fin, last;
    memset(&ca, 0, sizeof(ca));
    memset(&sum, 0, sizeof(sum));
    memset(&rm, 0, sizeof(rm));
    memset(&seqs, 0, sizeof(seqs));
    memset(&fin, 0, sizeof(fin));
    memset(&last, 0, sizeof(last));
    int M = 0, n_hi = 0, longest = 0, A = 0;
    for (int i = 0; i < V; ++i) {
        const PromptChunk& ch = chunks[i];
        ca.len[i] = rm.len[i] = ch.len;
        ca.off[i] = ch.tok;
        ca.before[i] = ch.before;
        rm.seq[i] = ch.b;
        rm.off[i] = M;
        M += ch.len;
        n_hi = std::max(n_hi, kv->len_hi[ch.b] + ch.before);
        longest = std::max(longest, ch.len);
        int a = 0;
        while (a < A && seqs.seq[a] != ch.b) ++a;
        if (a == A) seqs.seq[A++] = ch.b;
        sum.len[a] += ch.len;
    }
    const int n_fin = ending_rows(chunks, rm, &last, &fin), MB = prompt_blocks(M);
    launch_build_rows_chain(m->rt, tokens, ca, rm, m->rm_dev, kv->kv_len, V, Tp, hd, m->rope_freq, m->embed, 0, d, c.vocab, m->x, s);
    const RowRef rr = {m->rm_dev, 0};
    // (parts: what the partials' buffer holds)
    const AttnGeom ag = attn_geometry(nh, std::min(m->max_parts, m->MBmax * 32 * m->max_parts / (V * Tp)), V, Tp, n_hi, false);
    const bool whole = attn_whole_pays_prompt(Tp, n_hi);
    const int keep_A = V - keep, keep_TB = keep_Tp / 32;
    const size_t keep_stride = (size_t)keep_A * nh * keep_TB * 32 * hd;
    PartView prev = {nullptr, 0, d, nullptr, 0};
    for (int l = 0; l < c.n_layers; ++l) {
        const LayerW& lw = m->layers[l];
        launch_norm_pack(m->x, prev, lw.attn_norm, c.rms_eps, m->xn, nullptr, M, d, MB, nullptr, s);
        PartView pq = run_gemm(m, m->xn, lw.wqkv, m->part, M, MB, m->KBd, m->NBqkv, 3 * d, s);
        const KvSinks sinks = {kv->kc + l * kv->layer_stride, kv->vc + l * kv->layer_stride, kv->cap_blocks,
                               (uint16_t*)m->kt + l * keep_stride, (uint16_t*)m->vt + l * keep_stride, keep, keep_TB};
        launch_rope_kv(pq, m->rt, rr, m->q, m->ktp, m->vtp, V, Tp, nh, hd, s, &sinks);
        const int pa = prof_claim(m, PROF_ATTN, (double)V * (n_hi + Tp) * 2.0 * d * 2.0);
        if (whole)
            launch_attn_whole(m->q, sinks.kc, sinks.vc, m->ktp, m->vtp, kv->kv_len, m->rt.anc, m->attn_x, rr, V, nh, hd, Tp,
                              kv->cap_blocks, MB, s, prof_ev(m, pa, 0), prof_ev(m, pa, 1));
        else
            launch_tree_attn(m->q, sinks.kc, sinks.vc, m->ktp, m->vtp, kv->kv_len, m->rt.anc, m->opart, m->mlpart, rr, V, nh, hd, Tp,
                             kv->cap_blocks, ag.ncparts, ag.per, ag.tree_sep, s, prof_ev(m, pa, 0), prof_ev(m, pa, 1));
        if (!whole) launch_attn_merge(m->opart, m->mlpart, m->attn_x, rr, longest, V, nh, hd, Tp, ag.nparts, MB, s);
        PartView po = run_gemm(m, m->attn_x, lw.wo, m->part, M, MB, m->KBd, m->NBo, d, s);
        launch_norm_pack(m->x, po, lw.ffn_norm, c.rms_eps, m->xn, nullptr, M, d, MB, nullptr, s);
        const GemmPlan* gu = m->find_plan(MB, m->KBd, m->NBgu);
        const bool swiglu = gu && gemm_plan_swiglu(*gu);   // the projection sees whole sums: it leaves the next operand itself
        PartView pg = run_gemm(m, m->xn, lw.wgu, m->part, M, MB, m->KBd, m->NBgu, 2 * c.d_ffn, s, swiglu ? m->act : nullptr);
        if (!swiglu) launch_swiglu_pack(pg, c.d_ffn, m->Fpad, m->act, M, MB, s);
        prev = run_gemm(m, m->act, lw.wdown, m->part, M, MB, m->KBf, m->NBo, d, s);
    }
    launch_prefill_commit_setup(sum, seqs, A, Tp, kv->i_slots, kv->i_nacc, kv->n_old, kv->kv_len, m->fin_rows, n_fin, last, s);
    if (is_last) {                                         // (else a later pass of this call sets it)
        RowMap kr;
        ChainArgs kl;
        memset(&kr, 0, sizeof(kr));
        memset(&kl, 0, sizeof(kl));
        int kM = 0;
        for (int i = 0; i < keep_A; ++i) {
            kr.seq[i] = rm.seq[keep + i];
            kr.off[i] = kM;
            kl.len[i] = rm.len[keep + i];
            kM += kl.len[i];
        }
        m->scratch = scratch_of_pass(kv, kr, keep_A, kM, keep_Tp, kl.len, 0);
    }
    for (const PromptChunk& ch : chunks) kv->len_hi[ch.b] += ch.len;
    draft_from_prompts(m, kv, prev, n_fin, fin, s);
}

extern "C" int sd_prefill(sd_model* m, sd_kv* kv, const int32_t* tokens, const int32_t* lens, void* stream) {
    if (!m || !kv || !tokens || !lens) return fail(SD_ERR_NULL, "sd_prefill: NULL argument");
    if (kv->m != m) return fail(SD_ERR_STATE, "sd_prefill: cache belongs to another model");
    const int B = kv->B;
    hipStream_t s = (hipStream_t)stream;
    int Tp = (m->max_rows / B) / 32 * 32;
    if (Tp > 256) Tp = 256;                            // prompt chunks of up to 256 rows (the widest GEMM)
    if (Tp < 32) return fail(SD_ERR_SHAPE, "sd_prefill: max_rows %d too small for batch %d", m->max_rows, B);
    for (int b = 0; b < B; ++b) {
        if (lens[b] < 1) return fail(SD_ERR_SHAPE, "sd_prefill: every prompt needs at least one token");
        if (kv->len_hi[b] + lens[b] > kv->cap) return fail(SD_ERR_KV_FULL, "sd_prefill: sequence %d does not fit", b);
    }
    for (int rows = 32; rows <= 256; rows *= 2)            // every row count a pass can come down to
        if (pow2_blocks(rows) <= m->MBmax && !have_plans(m, rows, B, true, false))
            return fail(SD_ERR_STATE, "sd_prefill: no launch plan for %d rows (internal inconsistency)", rows);
    const std::vector<PromptPass> passes = cut_prompts(m, lens, B);
    size_t i = 0;
    for (int k : join_passes(m, passes)) {
        if (k > 1) run_prompt_passes(m, kv, tokens, &passes[i], k, i + k == passes.size(), s);
        else run_prompt_pass(m, kv, tokens, passes[i], s);
        i += k;
    }
    HIP_TRY(hipGetLastError());
    if (m->plan_missing) return fail(SD_ERR_STATE, "sd_prefill: a GEMM launch plan was missing");
    kv->has_draft = true;
    return SD_OK;
}

// ------------------------------------------------------------------------------------------ steps
static int step_common(sd_model* m, sd_kv* kv, uint64_t tree_uid, const int32_t* parent, const int32_t* depth,
                       const int32_t* rank, int T, int Tp, const uint32_t* stop_mask, sd_step_io* io, hipStream_t s,
                       const char* who, const sd_typical* ty = nullptr) {
    const sd_config& c = m->cfg;
    const int B = kv->B, H = c.n_medusa;
    if (kv->m != m) return fail(SD_ERR_STATE, "%s: cache belongs to another model", who);
    if (!kv->has_draft) return fail(SD_ERR_STATE, "%s: no draft state (call sd_prefill or sd_kv_set_draft first)", who);
    if (pow2_blocks(B * Tp) > m->MBmax)
        return fail(SD_ERR_SHAPE, "%s: %d rows exceed the model's max_rows", who, B * Tp);
    int n_hi = 0;
    for (int b = 0; b < B; ++b) {
        if (kv->len_hi[b] + H + 1 > kv->cap)
            return fail(SD_ERR_KV_FULL, "%s: sequence %d may exceed the cache (len <= %d, cap %d)", who, b,
                        kv->len_hi[b], kv->cap);
        n_hi = std::max(n_hi, kv->len_hi[b]);
    }
    const bool all_rows = m->draft_schedule == SD_DRAFT_ALL_NODES && T > 1 && !m->f32;   // (float32: one schedule only)
    const bool heads = T > 1 || m->greedy_drafts;      // plain greedy decoding may leave the draft heads out
    // rows of a sequence lie R apart: the tree's own nodes, no padding (see RowMap), except where the pass takes them
    // as [sequence][Tp]
    const int R = fused_eligible(m, B * Tp) ? Tp : T, M = B * R;
    RowMap rm;
    memset(&rm, 0, sizeof(rm));
    for (int b = 0; b < B; ++b) { rm.off[b] = b * R; rm.len[b] = R; rm.seq[b] = b; }
    if (!have_plans(m, M, B, heads, all_rows))
        return fail(SD_ERR_STATE, "%s: no launch plan for %d rows (internal inconsistency)", who, M);
    int32_t* n_accept = io->n_accept ? io->n_accept : kv->i_nacc;
    int32_t* tokens = io->tokens ? io->tokens : kv->i_tokens;
    int32_t* slots = io->src_slots ? io->src_slots : kv->i_slots;
    const int32_t* cand = io->forced_cand ? io->forced_cand : kv->cand;

    const PassGeom ag = pass_geometry(m, kv, nullptr, B, M, Tp, n_hi);
    const ScratchRows scratch = scratch_of_pass(kv, rm, B, M, Tp, nullptr, T);
    auto enqueue = [&](hipStream_t s) {
    launch_build_rows_tree(m->rt, parent, depth, rank, kv->root_tok, cand, kv->kv_len, B, T, Tp, R, H, c.topk, c.head_dim,
                           m->rope_freq, m->embed, m->f32 ? 1 : 0, c.d_model, c.vocab, m->x, s);
    // the logits somebody reads: the caller's dense rows [b][T][V], or (sampling decoding alone) the padded ones
    const bool dense = R == T || B == 1;
    float* lg = io->logits && dense ? io->logits : (io->logits || ty) ? m->logits : nullptr;
    const int ldl = lg == m->logits ? m->Vpad : c.vocab;
    // plain decoding drafts from the only row a sequence has: one pass of the LM head for its base and head rows
    const bool known = T == 1 && dense && heads && !fused_eligible(m, B * Tp);
    PartView pl = run_forward(m, kv, rm, B, M, R, Tp, n_hi, ag, !known, all_rows, s);
    if (known) {
        run_known_rows(m, kv, pl, B, nullptr, every_sequence(), lg, ldl, io->head_logits, s);
    } else {
        launch_rank_best(pl, 0, dense ? B * T : M, c.vocab, lg, ldl, m->best, s);
        if (io->logits && !dense)
            for (int b = 0; b < B; ++b)
                launch_rank_best(pl, b * R, T, c.vocab, io->logits + (size_t)b * T * c.vocab, c.vocab,
                                 m->best + (size_t)b * R * rank_chunks(c.vocab), s);
    }
    VerifyArgs va;
    va.parent = parent; va.depth = depth; va.T = T; va.H = H; va.fallback = c.trunc_fallback;
    va.src_stride = R; va.Tp = R; va.V = c.vocab;
    va.tok = m->rt.tok; va.am = nullptr; va.best = m->best; va.n_chunks = rank_chunks(c.vocab); va.am_out = io->argmax;
    va.stop_mask = stop_mask;
    va.n_accept = n_accept; va.n_accept_raw = io->n_accept_raw; va.tokens = tokens; va.src_slots = slots;
    va.kv_len = kv->kv_len; va.n_old = kv->n_old; va.root_tok = kv->root_tok; va.last_row = kv->last_row;
    va.logits = nullptr; va.ld = 0; va.row_stats = nullptr; va.inv_temperature = 1.f;
    if (ty) {
        va.inv_temperature = 1.f / ty->temperature;
        launch_row_stats(lg, ldl, c.vocab, m->row_stats, B, T, R, va.inv_temperature, ty->epsilon,
                         ty->delta, s);
        if (ty->row_stats) launch_copy_row_stats(m->row_stats, (float4*)ty->row_stats, B, T, R, s);
        va.logits = lg; va.ld = ldl; va.row_stats = m->row_stats;
    }
    launch_verify(va, B, s);
    if (ty)      // the next root is drawn from the base distribution at the last kept node
        launch_sample_root(lg, ldl, c.vocab, kv->last_row, ty->u, va.inv_temperature, kv->root_tok, B,
                           M, s);
    commit_rows(m, kv, scratch, false, slots, n_accept, H + 1, s);
    if (all_rows) run_draft_heads_all_rows(m, kv, B, M, io->head_logits, s);
    else if (heads && !known) run_draft_heads(m, kv, B, io->head_logits, s);
    };

    if (m->use_graphs && !m->prof.on && !ty) {
        // everything the launch sequence depends on besides device-resident state
        std::vector<uint64_t> key = {kv->uid, tree_uid, (uint64_t)(uintptr_t)parent, (uint64_t)T, (uint64_t)Tp,
                                     (uint64_t)ag.ncparts, (uint64_t)ag.per, (uint64_t)ag.tree_sep, (uint64_t)ag.whole,
                                     (uint64_t)(uintptr_t)stop_mask,
                                     (uint64_t)(uintptr_t)n_accept, (uint64_t)(uintptr_t)tokens,
                                     (uint64_t)(uintptr_t)slots, (uint64_t)(uintptr_t)io->n_accept_raw,
                                     (uint64_t)(uintptr_t)io->logits, (uint64_t)(uintptr_t)io->argmax,
                                     (uint64_t)(uintptr_t)io->head_logits, (uint64_t)(uintptr_t)cand,
                                     (uint64_t)m->draft_schedule, (uint64_t)heads,
                                     (uint64_t)(m->use_fused ? 1 : 0) | ((uint64_t)m->sync_timeout_ticks << 1),
                                     (uint64_t)(uintptr_t)m->timeline, (uint64_t)m->timeline_launches};
        key.insert(key.end(), ag.split.slot, ag.split.slot + ag.split.n);
        hipGraphExec_t exec = nullptr;
        for (const sd_model::StepGraph& g : m->graphs)
            if (g.key == key) { exec = g.exec; break; }
        if (!exec) {
            if (m->graphs.size() >= 64) {              // bounded cache: start over
                for (sd_model::StepGraph& g : m->graphs) hipGraphExecDestroy(g.exec);
                m->graphs.clear();
            }
            hipGraph_t graph = nullptr;
            if (!m->cap_stream) HIP_TRY(hipStreamCreateWithFlags(&m->cap_stream, hipStreamNonBlocking));
            HIP_TRY(hipStreamBeginCapture(m->cap_stream, hipStreamCaptureModeThreadLocal));
            enqueue(m->cap_stream);
            hipError_t e = hipStreamEndCapture(m->cap_stream, &graph);
            if (e != hipSuccess) return fail(SD_ERR_HIP, "%s: graph capture failed: %s", who, hipGetErrorString(e));
            e = hipGraphInstantiate(&exec, graph, nullptr, nullptr, 0);
            hipGraphDestroy(graph);
            if (e != hipSuccess) return fail(SD_ERR_HIP, "%s: hipGraphInstantiate: %s", who, hipGetErrorString(e));
            m->graphs.push_back({key, exec});
        }
        HIP_TRY(hipGraphLaunch(exec, s));
    } else {
        enqueue(s);
    }
    m->scratch = scratch;                              // (of a replayed step too: passes may have run since its capture)
    HIP_TRY(hipGetLastError());
    if (m->plan_missing) return fail(SD_ERR_STATE, "%s: a GEMM launch plan was missing", who);
    for (int b = 0; b < B; ++b) kv->len_hi[b] += (T == 1) ? 1 : H + 1;
    return SD_OK;
}

extern "C" int sd_spec_step(sd_model* m, sd_kv* kv, const sd_tree* tree, const uint32_t* stop_mask, sd_step_io* io,
                            void* stream) {
    if (!m || !kv || !tree || !stop_mask || !io) return fail(SD_ERR_NULL, "sd_spec_step: NULL argument");
    if (tree->H != m->cfg.n_medusa || tree->topk != m->cfg.topk)
        return fail(SD_ERR_BAD_TREE, "sd_spec_step: tree was built for %d heads / top-%d", tree->H, tree->topk);
    return step_common(m, kv, tree->uid, tree->parent, tree->depth, tree->rank, tree->T, tree->Tp, stop_mask, io,
                       (hipStream_t)stream, "sd_spec_step");
}

// Commit stage alone: rows of the tree scratch, as the last pass over this cache's batch left them, appended to
// every sequence.
extern "C" int sd_kv_commit_rows(sd_model* m, sd_kv* kv, const int32_t* src_slots, const int32_t* n_rows, int32_t width,
                                 void* stream) {
    if (!m || !kv || !src_slots || !n_rows) return fail(SD_ERR_NULL, "sd_kv_commit_rows: NULL argument");
    if (kv->m != m) return fail(SD_ERR_STATE, "sd_kv_commit_rows: cache belongs to another model");
    if (m->scratch.B != kv->B || m->scratch.Tp < 32)
        return fail(SD_ERR_STATE, "sd_kv_commit_rows: no pass over a batch of %d has left tree rows to commit", kv->B);
    if (width < 1 || width > m->scratch.Tp)
        return fail(SD_ERR_SHAPE, "sd_kv_commit_rows: width must be in 1..%d (the rows of the last pass)", m->scratch.Tp);
    for (int b = 0; b < kv->B; ++b)
        if (kv->len_hi[b] + width > kv->cap)
            return fail(SD_ERR_KV_FULL, "sd_kv_commit_rows: sequence %d may exceed the cache (len <= %d, cap %d)", b,
                        kv->len_hi[b], kv->cap);
    hipStream_t s = (hipStream_t)stream;
    uint32_t held = 0;                                 // a sequence that the pass did not hold has no rows to commit
    for (int i = 0; i < m->scratch.n; ++i) held |= 1u << m->scratch.seq[i];
    launch_commit_setup(n_rows, width, held, kv->B, kv->i_nacc, kv->n_old, kv->kv_len, s);
    commit_rows(m, kv, m->scratch, true, src_slots, kv->i_nacc, width, s);
    HIP_TRY(hipGetLastError());
    for (int b = 0; b < kv->B; ++b)
        if ((held >> b) & 1u) kv->len_hi[b] += width;
    return SD_OK;
}

static int check_typical(float temperature, float epsilon, float delta, const char* who) {
    if (!(temperature > 0.f) || !std::isfinite(temperature))
        return fail(SD_ERR_SHAPE, "%s: temperature must be positive and finite", who);
    if (!(epsilon >= 0.f && epsilon <= 1.f) || !(delta >= 0.f) || !std::isfinite(delta))
        return fail(SD_ERR_SHAPE, "%s: need 0 <= epsilon <= 1 and 0 <= delta < inf", who);
    return SD_OK;
}

extern "C" int sd_spec_step_typical(sd_model* m, sd_kv* kv, const sd_tree* tree, const uint32_t* stop_mask,
                                    sd_step_io* io, const sd_typical* ty, void* stream) {
    if (!m || !kv || !tree || !stop_mask || !io || !ty) return fail(SD_ERR_NULL, "sd_spec_step_typical: NULL argument");
    if (tree->H != m->cfg.n_medusa || tree->topk != m->cfg.topk)
        return fail(SD_ERR_BAD_TREE, "sd_spec_step_typical: tree was built for %d heads / top-%d", tree->H, tree->topk);
    if (!ty->u) return fail(SD_ERR_NULL, "sd_spec_step_typical: sd_typical.u is NULL");
    if (int rc = check_typical(ty->temperature, ty->epsilon, ty->delta, "sd_spec_step_typical")) return rc;
    return step_common(m, kv, tree->uid, tree->parent, tree->depth, tree->rank, tree->T, tree->Tp, stop_mask, io,
                       (hipStream_t)stream, "sd_spec_step_typical", ty);
}

extern "C" int sd_greedy_step(sd_model* m, sd_kv* kv, sd_step_io* io, void* stream) {
    if (!m || !kv || !io) return fail(SD_ERR_NULL, "sd_greedy_step: NULL argument");
    return step_common(m, kv, 0, m->g_parent, m->g_depth, m->g_rank, 1, 32, m->zero_stop, io, (hipStream_t)stream,
                       "sd_greedy_step");
}

extern "C" int sd_verify_tree(const sd_tree* tree, int32_t batch, int32_t n_medusa, int32_t trunc_fallback,
                              int32_t vocab, const int32_t* tok, const int32_t* am, const uint32_t* stop_mask,
                              int32_t* n_accept, int32_t* n_accept_raw, int32_t* tokens, int32_t* src_slots,
                              void* stream) {
    if (!tree || !tok || !am || !stop_mask || !n_accept || !tokens || !src_slots)
        return fail(SD_ERR_NULL, "sd_verify_tree: NULL argument");
    if (batch < 1 || batch > 65535) return fail(SD_ERR_SHAPE, "sd_verify_tree: bad batch");
    if (n_medusa != tree->H) return fail(SD_ERR_BAD_TREE, "sd_verify_tree: tree was built for %d heads", tree->H);
    if (trunc_fallback != SD_TRUNC_KEEP_ALL && trunc_fallback != SD_TRUNC_KEEP_ONE)
        return fail(SD_ERR_SHAPE, "sd_verify_tree: bad trunc_fallback");
    VerifyArgs va;
    memset(&va, 0, sizeof(va));
    va.parent = tree->parent; va.depth = tree->depth; va.T = tree->T; va.H = tree->H; va.fallback = trunc_fallback;
    va.src_stride = tree->T; va.Tp = tree->Tp; va.V = vocab;
    va.tok = tok; va.am = am; va.stop_mask = stop_mask;
    va.n_accept = n_accept; va.n_accept_raw = n_accept_raw; va.tokens = tokens; va.src_slots = src_slots;
    launch_verify(va, batch, (hipStream_t)stream);
    HIP_TRY(hipGetLastError());
    return SD_OK;
}

extern "C" int sd_verify_tree_typical(const sd_tree* tree, int32_t batch, int32_t n_medusa, int32_t trunc_fallback,
                                      int32_t vocab, const int32_t* tok, const float* logits, float temperature,
                                      float epsilon, float delta, const uint32_t* stop_mask, float* row_stats,
                                      int32_t* n_accept, int32_t* n_accept_raw, int32_t* tokens, int32_t* src_slots,
                                      void* stream) {
    if (!tree || !tok || !logits || !stop_mask || !row_stats || !n_accept || !tokens || !src_slots)
        return fail(SD_ERR_NULL, "sd_verify_tree_typical: NULL argument");
    if (batch < 1 || batch > 65535) return fail(SD_ERR_SHAPE, "sd_verify_tree_typical: bad batch");
    if (vocab < 1 || vocab > 163840) return fail(SD_ERR_SHAPE, "sd_verify_tree_typical: bad vocab");
    if (n_medusa != tree->H) return fail(SD_ERR_BAD_TREE, "sd_verify_tree_typical: tree was built for %d heads", tree->H);
    if (trunc_fallback != SD_TRUNC_KEEP_ALL && trunc_fallback != SD_TRUNC_KEEP_ONE)
        return fail(SD_ERR_SHAPE, "sd_verify_tree_typical: bad trunc_fallback");
    if (int rc = check_typical(temperature, epsilon, delta, "sd_verify_tree_typical")) return rc;
    hipStream_t s = (hipStream_t)stream;
    const int T = tree->T;
    launch_row_stats(logits, vocab, vocab, (float4*)row_stats, batch, T, T, 1.f / temperature, epsilon, delta, s);
    VerifyArgs va;
    memset(&va, 0, sizeof(va));
    va.parent = tree->parent; va.depth = tree->depth; va.T = T; va.H = tree->H; va.fallback = trunc_fallback;
    va.src_stride = T; va.Tp = tree->Tp; va.V = vocab;
    va.tok = tok; va.am = tok; va.stop_mask = stop_mask;      // (am decides nothing under typical acceptance; it is read, so it must be readable)
    va.n_accept = n_accept; va.n_accept_raw = n_accept_raw; va.tokens = tokens; va.src_slots = src_slots;
    va.logits = logits; va.ld = vocab; va.row_stats = (const float4*)row_stats; va.inv_temperature = 1.f / temperature;
    launch_verify(va, batch, s);
    HIP_TRY(hipGetLastError());
    return SD_OK;
}

// ------------------------------------------------------------------------------------------ no allocation
// Per-node statistics of sd_verify_tree_typical_static: one copy per GPU, held until the process ends.
#define SD_STATIC_ROWS 4096
static __device__ __align__(256) float4 scratch[SD_STATIC_ROWS];
// Device address of `scratch` on every GPU this process has used it on. The array's name is only a host-side
// handle: the address a kernel can use comes from hipGetSymbolAddress, per device.
#define SD_MAX_DEVICES 64
static float4* g_scratch_dev[SD_MAX_DEVICES] = {};

static int static_scratch(float4** out) {
    int dev = -1;
    HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= SD_MAX_DEVICES) return fail(SD_ERR_SHAPE, "device ordinal %d not supported", dev);
    float4* p = __atomic_load_n(&g_scratch_dev[dev], __ATOMIC_ACQUIRE);
    if (!p) {                                          // first call on this device (two racing threads get the same answer)
        void* addr = nullptr;
        HIP_TRY(hipGetSymbolAddress(&addr, HIP_SYMBOL(scratch)));
        if (!addr) return fail(SD_ERR_HIP, "hipGetSymbolAddress returned no address");
        p = (float4*)addr;
        __atomic_store_n(&g_scratch_dev[dev], p, __ATOMIC_RELEASE);
    }
    *out = p;
    return SD_OK;
}

extern "C" int sd_verify_tree_typical_static(const sd_tree* tree, int32_t batch, int32_t n_medusa,
                                             int32_t trunc_fallback, int32_t vocab, const int32_t* tok,
                                             const float* logits, float temperature, float epsilon, float delta,
                                             const uint32_t* stop_mask, int32_t* n_accept, int32_t* n_accept_raw,
                                             int32_t* tokens, int32_t* src_slots, void* stream) {
    if (!tree || !tok || !logits || !stop_mask || !n_accept || !tokens || !src_slots)
        return fail(SD_ERR_NULL, "sd_verify_tree_typical_static: NULL argument");
    if (batch < 1 || batch > 65535) return fail(SD_ERR_SHAPE, "sd_verify_tree_typical_static: bad batch");
    if ((int64_t)batch * tree->T > SD_STATIC_ROWS)
        return fail(SD_ERR_SHAPE, "sd_verify_tree_typical_static: batch * tree nodes = %lld exceeds the %d rows of the "
                    "static statistics buffer (use sd_verify_tree_typical with a buffer of your own)",
                    (long long)batch * tree->T, SD_STATIC_ROWS);
    if (vocab < 1 || vocab > 163840) return fail(SD_ERR_SHAPE, "sd_verify_tree_typical_static: bad vocab");
    if (n_medusa != tree->H)
        return fail(SD_ERR_BAD_TREE, "sd_verify_tree_typical_static: tree was built for %d heads", tree->H);
    if (trunc_fallback != SD_TRUNC_KEEP_ALL && trunc_fallback != SD_TRUNC_KEEP_ONE)
        return fail(SD_ERR_SHAPE, "sd_verify_tree_typical_static: bad trunc_fallback");
    if (int rc = check_typical(temperature, epsilon, delta, "sd_verify_tree_typical_static")) return rc;
    float4* stats = nullptr;
    if (int rc = static_scratch(&stats)) return rc;
    hipStream_t s = (hipStream_t)stream;
    const int T = tree->T;
    // every row of the statistics that the acceptance kernel reads is written first by this launch, so nothing
    // of the previous call's contents needs clearing
    launch_row_stats(logits, vocab, vocab, stats, batch, T, T, 1.f / temperature, epsilon, delta, s);
    VerifyArgs va;
    memset(&va, 0, sizeof(va));
    va.parent = tree->parent; va.depth = tree->depth; va.T = T; va.H = tree->H; va.fallback = trunc_fallback;
    va.src_stride = T; va.Tp = tree->Tp; va.V = vocab;
    va.tok = tok; va.am = tok; va.stop_mask = stop_mask;      // (am decides nothing under typical acceptance; it is read, so it must be readable)
    va.n_accept = n_accept; va.n_accept_raw = n_accept_raw; va.tokens = tokens; va.src_slots = src_slots;
    va.logits = logits; va.ld = vocab; va.row_stats = stats; va.inv_temperature = 1.f / temperature;
    launch_verify(va, batch, s);
    HIP_TRY(hipGetLastError());
    return SD_OK;
}

extern "C" int sd_sample_tokens(const float* logits, int32_t n_rows, int32_t ld, int32_t vocab, const int32_t* rows,
                                const float* u, int32_t n, float temperature, int32_t* out, void* stream) {
    if (!logits || !rows || !u || !out) return fail(SD_ERR_NULL, "sd_sample_tokens: NULL argument");
    if (n < 1 || n > 65535 || n_rows < 1) return fail(SD_ERR_SHAPE, "sd_sample_tokens: bad n");
    if (vocab < 1 || vocab > 163840 || ld < vocab) return fail(SD_ERR_SHAPE, "sd_sample_tokens: bad vocab / ld");
    if (!(temperature > 0.f) || !std::isfinite(temperature))
        return fail(SD_ERR_SHAPE, "sd_sample_tokens: temperature must be positive and finite");
    launch_sample_root(logits, ld, vocab, rows, u, 1.f / temperature, out, n, n_rows, (hipStream_t)stream);
    HIP_TRY(hipGetLastError());
    return SD_OK;
}
