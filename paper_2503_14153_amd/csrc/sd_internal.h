// Internal declarations shared by the HIP translation units of libspecdec (gfx950 only).
//
// Memory layouts (all "fragment" layouts are chosen so that one wave64 load instruction of
// 16 bytes per lane fetches one contiguous 1 KiB MFMA operand of v_mfma_f32_32x32x16_bf16:
// lane l supplies row/column (l % 32) and the eight contraction elements g*8 .. g*8+7 with
// g = l / 32):
//
//   packed activation  X[kb][mb][part][lane][8]  element (row m, col k): kb = k/16, mb = m/32,
//                                            lane = m%32 + 32*((k/8)&1), slot = k%8;
//                                            part 0 = bf16(x), part 1 = bf16(x - part 0): the
//                                            activations enter the MFMAs as a two-term bf16
//                                            expansion (about 16 mantissa bits), see gemm.hip
//   packed weight      W[kb][nb][lane][8]    element (out n, in k):  nb = n/32, kb = k/16,
//                                            lane = n%32 + 32*((k/8)&1), slot = k%8
//   key block (32 rows of one head)          K[kk][lane][8]: row c, dim e: kk = e/16,
//                                            lane = c%32 + 32*((e/8)&1), slot = e%8
//   value block (32 rows of one head)        V[p][eb][lane][8]: row c, dim e: p = (c%32)/16,
//                                            eb = e/32, lane = e%32 + 32*((c/4)&1),
//                                            slot = 4*((c/8)&1) + c%4
//     (the value rows are permuted inside a block so that the softmax probabilities, as they
//      come out of the QK^T accumulator, are already the B operand of the PV product)
#pragma once
#include <hip/hip_runtime.h>
#include <hip/hip_ext.h>
#include <stdint.h>
#include <stddef.h>

#include "../../include/specdec.h"
#include "gemm_plan.h"

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

#ifdef __HIPCC__
// two-term bf16 expansion of eight floats: hi = bf16(f), lo = bf16(f - hi)
static __device__ inline void split_hilo(const float (&f)[8], bf16x8& hi, bf16x8& lo) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        __bf16 h = (__bf16)f[i];
        hi[i] = h;
        lo[i] = (__bf16)(f[i] - (float)h);
    }
}
#endif

#define SD_MAX_TREE 256
#define SD_ANC_WORDS 8

// element index of (row m, col k) in part 0 of a packed activation; part 1 is XPART further
#define XPART 512
static __host__ __device__ inline size_t xpack_index(int m, int k, int MB) {
    int kb = k >> 4, g = (k >> 3) & 1, s = k & 7, mb = m >> 5, r = m & 31;
    return ((((size_t)kb * MB + mb) * 2 * 64) + (size_t)(r + 32 * g)) * 8 + s;
}
// same for a query block: Q[kk][part][lane][8] per 32 queries of one head
static __host__ __device__ inline size_t qblk_index(int t, int e, int HD) {
    int blk = t >> 5, r = t & 31, kk = e >> 4, g = (e >> 3) & 1, s = e & 7;
    return (size_t)blk * (64 * HD) + ((size_t)(kk * 2 * 64 + r + 32 * g)) * 8 + s;
}
// offset (in elements) of (row c, dim e) inside a head's key blocks; HD = head_dim
static __host__ __device__ inline size_t kblk_index(int c, int e, int HD) {
    int blk = c >> 5, r = c & 31, kk = e >> 4, g = (e >> 3) & 1, s = e & 7;
    return (size_t)blk * (32 * HD) + ((size_t)(kk * 64 + r + 32 * g)) * 8 + s;
}
static __host__ __device__ inline size_t vblk_index(int c, int e, int HD) {
    int blk = c >> 5, cc = c & 31, p = cc >> 4, g = (cc >> 2) & 1, s = ((cc >> 3) & 1) * 4 + (cc & 3);
    int eb = e >> 5, er = e & 31;
    return (size_t)blk * (32 * HD) + ((size_t)((p * (HD / 32) + eb) * 64 + er + 32 * g)) * 8 + s;
}

// ---- per-call row table (device) -----------------------------------------------------------
// The M rows of a pass are packed: sequence i of the pass owns rows [off[i], off[i] + len[i]) of the residual stream, of
// every GEMM operand and of every partial sum, with no padding between sequences, so eight sequences of plain decoding
// are 8 rows and not 256 (7B shape, GEMM launches per layer 232 -> 86 us). Only attention works on 32-row blocks per
// sequence: its queries, the tree's K/V scratch and its partials are [i][Tp], row t there is packed row off[i] + t for
// t < len[i] and padding (never read back as a result) beyond. (float32 path: the scratch is packed too.)
#define SD_MAX_BATCH 32
struct RowMap {
    int32_t off[SD_MAX_BATCH], len[SD_MAX_BATCH];   // len >= 1
    int32_t seq[SD_MAX_BATCH];                      // sequence of the cache
};
struct SeqList { int32_t seq[SD_MAX_BATCH]; };      // one number per sequence of a pass
// The map of a prompt pass in device memory. ctx: rows that sequence i's rows attend besides their own (the committed ones,
// and the sequence's rows earlier in the same pass, which are in the cache by the time attention runs).
struct PassMap { int32_t off[SD_MAX_BATCH], len[SD_MAX_BATCH], seq[SD_MAX_BATCH], ctx[SD_MAX_BATCH]; };
// What the kernels of a layer get: every sequence of a step has the same number of rows, R (map NULL); a prompt pass leaves
// its map in device memory. (As an argument of every launch the map's 384 bytes cost the 64-node step 1 %, read from
// memory by every launch another 1 %: the attention launch's first addresses wait for it, 14.9 -> 15.5 us.)
struct RowRef {
    const PassMap* map;
    int R;
#ifdef __HIPCC__
    __device__ __forceinline__ int off(int i) const { return map ? map->off[i] : i * R; }
    __device__ __forceinline__ int len(int i) const { return map ? map->len[i] : R; }
    __device__ __forceinline__ int seq(int i) const { return map ? map->seq[i] : i; }
#endif
};
struct RowTable {
    int32_t* tok;      // [M] token id of every row (0 for padding rows)
    int32_t* pos;      // [M] position
    uint32_t* anc;     // [i][Tp][SD_ANC_WORDS] bit j set: row may attend tree row j of its sequence
    float2* cs;        // [M][head_dim/2] (cos, sin) of the rotary angle
};

// Partial results of a GEMM whose contraction was divided over several workgroups: the
// consumer sums `count(col)` slots. cnt == NULL means every column has nmax slots.
struct PartView {
    const float* base;
    size_t slot_stride;      // floats between slots
    int ld;                  // floats between rows
    const int32_t* cnt;      // [ceil(ld / 256)] slots per 256-column group, or NULL
    int nmax;
};
#ifdef __HIPCC__
static __device__ inline int part_count(const PartView& p, int col) { return p.cnt ? p.cnt[col >> 8] : p.nmax; }
#endif

// The launch before a GEMM has just written its activations: the first workgroup of an XCD that asks for a line of them waits for
// memory, and since the workgroups of a segment walk in step, each does so at every step. So the workgroups that share an
// XCD (they are dealt round-robin) and a segment fetch the segment's lines together at the start, one line per thread, while
// the first weights are on their way; the loads of the walk then find them in L2. (Another mapping only costs time.)
// k_gemm_sk only: steps of four layers at 64 rows 724.5 -> 719 us, five 12-node trees 770 -> 761, 16 k rows 907 -> 899. Level or
// slower for k_gemm_kw (16 rows 553 -> 554) and for the 256-row kernel (1286 -> 1310: four times the lines).
struct OperandTouch { uint32_t magic; int shares; };   // ceil(2^32 / period), workgroups of an XCD and a segment
static inline OperandTouch operand_touch(int G, int S) {
    int period = 8;
    while (period % S) period += 8;                    // (workgroup g: XCD g % 8, segment g % S)
    return OperandTouch{(uint32_t)((0x100000000ull + period - 1) / period), (G + period - 1) / period};
}
#ifdef __HIPCC__
static __device__ __forceinline__ uint32_t touch_operand(const void* slice, int bytes, OperandTouch t) {
    const int lines = bytes >> 7, l = (int)__umulhi(blockIdx.x, t.magic) + t.shares * (int)threadIdx.x;
    return *(const uint32_t*)((const char*)slice + ((size_t)min(l, lines - 1) << 7));
}
static __device__ __forceinline__ void touched(uint32_t v) { asm volatile("" ::"v"(v)); }     // (keeps the load)
#endif

// Rows whose RMSNorm scale is applied AFTER the contraction (the operand holds x * gain, see row_ops.h):
// ssq [ceil(n_parts / 4)][Mp][4] partial sums of squares of every row (Mp = the GEMM's padded row count, part p of
// row m at ((p / 4) * Mp + m) * 4 + p % 4; parts beyond n_parts are zero); every output of row m is multiplied by
// 1 / sqrt(sum_p ssq[p][m] * inv_d + eps).
struct SkRowScale {
    const float* ssq;        // NULL: no scaling
    int n_parts;
    float inv_d, eps;
};

// ---- the persistent layer kernel (fused.hip) -----------------------------------------------
// One weight-streaming GEMM as a phase: its plan, operands and the buffer of its partial sums.
struct FusedGemm {
    const bf16x8* X;         // packed activations (written by an earlier phase of the same launch)
    const bf16x8* W;         // packed weights
    float* out;              // partial sums [slot][row][col]
    size_t slot_stride;
    int KB, NB, ldo, upw, rem, G, nmax;
    uint32_t kb_magic;
    const int32_t* slot0;    // [G]
    const int32_t* cnt;      // [NG] or NULL (nmax slots everywhere)
    SkRowScale sc;           // deferred RMS scale of the rows (the GEMMs that follow a norm), or ssq NULL
};
struct FusedSync {
    unsigned* counters;      // this launch's barrier counters: 9 words 256 bytes apart, zero at launch
    unsigned* abort_flag;    // set to 1 by a workgroup whose wait ran out
    unsigned long long timeout_ticks;   // of the 100 MHz real-time counter
};
// what a launch runs, in this order; each GEMM comes with the row-wise phase that produces its operand
enum {
    FUSED_GEMM_O = 1,        // merge of the attention parts, O projection
    FUSED_GEMM_GU = 2,       // residual + norm (feed-forward), gate/up projection
    FUSED_GEMM_DN = 4,       // SwiGLU, down projection
    FUSED_GEMM_Q = 8,        // residual + norm (attention, or the final one), QKV projection or LM head
    FUSED_ROPE = 16          // rotary embedding and the tree K/V write
};
#define FUSED_SYNC_WORDS 1024    // counters of one launch (9 used, spaced 64 words)
struct FusedArgs {
    uint32_t phases;         // FUSED_* bits
    int M, MB, B, Tp, d, nh, hd, F, Fpad, nparts;
    float eps;
    float* x;                // residual stream [M][d]
    const float* opart; const float2* mlpart;      // attention parts (merge)
    bf16x8* att;             // merged attention output, operand of g_o
    FusedGemm g_o, g_gu, g_dn, g_q;
    const uint16_t* gain_f; bf16x8* xn_f; float* ssq_f;   // norm before the feed-forward block -> operand of g_gu
    bf16x8* act;             // SwiGLU output, operand of g_dn
    const uint16_t* gain_a; bf16x8* xn_a; float* ssq_a;   // norm before attention (or the final norm) -> operand of g_q
    PartView prev;           // what NORM_A adds when the launch starts with it
    RowTable rt; bf16x8* q; uint16_t* kt; uint16_t* vt;   // rotary phase outputs
    const bf16x8* zfrag;
    FusedSync sync;
    unsigned long long* timeline;   // NULL, or [24][gridDim.x] time stamps (100 MHz): entry to each phase, end of launch
};

#define SD_MAX_MEDUSA 15
// prompt tokens of every sequence of the pass; before: rows of the same sequence earlier in this pass
struct ChainArgs { int32_t off[SD_MAX_BATCH]; int32_t len[SD_MAX_BATCH]; int32_t before[SD_MAX_BATCH]; };
// Where the rotary stage of a prompt pass of several chunks puts keys and values besides the pass's own scratch: the cache
// (one layer's planes), and for sequences keep .. of the pass the scratch that a later commit reads ([i - keep][keep_TB blocks]).
struct KvSinks { uint16_t *kc, *vc; int cap_blocks; uint16_t *kk, *vk; int keep, keep_TB; };
struct MedusaBias { const uint16_t* p[SD_MAX_MEDUSA + 1]; };
struct VerifyArgs {
    const int32_t *parent, *depth;      // device tree tables [T]
    int T, H, fallback, src_stride, Tp, V;
    const int32_t *tok, *am;            // [B][src_stride]; am not read when best is given
    const float2* best;                 // NULL, or [B][src_stride][n_chunks] (launch_rank_best)
    int n_chunks;
    int32_t* am_out;                    // [B][T] or NULL: the arg-max of every node
    const uint32_t* stop_mask;
    int32_t *n_accept, *n_accept_raw, *tokens, *src_slots;   // outputs, [B] / [B][H+1]
    int32_t *kv_len, *n_old, *root_tok, *last_row;           // carried state, may be NULL
    // typical acceptance (sampling decoding) instead of greedy when row_stats != NULL
    const float* logits;                // [B*Tp][ld]
    int ld;
    const float4* row_stats;            // [B*Tp]: {max logit, Z, entropy, c = log(threshold * Z)} per row
    float inv_temperature;
};

// ---- launchers (defined in the kernel translation units) ----------------------------------
// All take a stream; all sizes have been validated by the caller.
void launch_pack_weight(const void* src, void* dst, int N, int K, int nb_offset, int NBdst, int KB, hipStream_t s);
// fills every field of the plan except cnt_dev; cnt_host receives the per-group counts
// cnt_host [>= ceil(NB/8)] and slot0_host [>= 256] receive the tables the device copies hold
void gemm_plan_make(GemmPlan* p, int MB, int KB, int NB, int32_t* cnt_host, int32_t* slot0_host);
// out must hold plan.slots * (MB*32) * (NB*32) floats; zfrag: 2 KiB of zeros (device);
// returns the view consumers read
// ev0 / ev1 (both or neither): events that receive the kernel's own start and end time stamps,
// for per-kernel timing without launch gaps
// sc: deferred RMS scale of the rows (ssq NULL: none; not available at four row blocks)
// rows: rows that exist; the partial tiles' other rows are not written
PartView launch_gemm(const GemmPlan& p, const void* Xp, const void* Wp, const void* zfrag, float* out, int rows, hipStream_t s,
                     hipEvent_t ev0 = nullptr, hipEvent_t ev1 = nullptr, void* swiglu = nullptr, int swiglu_KB = 0);
// A handful of rows (few.hip): float32 rows in, every column finished by one workgroup, no partial sums.
struct FewLinear {
    const float* X; int ldx;                                          // rows [M][ldx] (row m: gather[m] if given)
    const int32_t* gather;
    const bf16x8* Xp;                                                 // or the ready-made operand (add), M <= FEW_LAYER_ROWS
    const uint16_t* gain; float eps;                                  // RMSNorm of the rows, or NULL
    const bf16x8* W; int KB, NB;                                        // packed weights, KB * NB KiB < 4 GiB
    int M, n_units;                                                   // M <= FEW_ROWS; columns / 16 (pairs, if gate and up)
    int up;                                                           // first up block, in units of 16 columns
    float* out; int ldo;
    bf16x8* packed; int MB;                                           // results as an operand instead: swiglu: ready-made for
                                                                      // add; heads (or NULL): of a GEMM of MB row blocks
    const float* row_scale;                                           // store: factor of every row's result, or NULL
    int base; float* scale_out;                                       // heads: 1 = the rows h themselves come first, as x * gain
                                                                      // whose factor goes to scale_out (heads' rows: 1), so that
                                                                      // their products are the bits that norm(X) gives
    const float* opart; const float2* mlpart;                         // or NULL: the rows are the merged attention parts,
    int nh, hd, Tp, nparts, R;                                        // row m = b * R + t; few_merges(M, d)
    int own[2];                                                       // parts of sequence b (of nparts)
};
#define FEW_ROWS 16
#define FEW_LAYER_ROWS 8         // layers (add, swiglu): one product takes both terms
#define FEW_MERGE_ROWS 2         // (every workgroup merges all of the rows, 8 bytes of LDS per input)
// d: 48 KiB of operand beside 17.5 KiB of sums at most, of the 160 KiB that a workgroup may ask for (tested to 6144)
static inline bool few_merges(int M, int d) { return M <= FEW_MERGE_ROWS && d <= 6144; }
// 16-byte unit of (row m, inputs 8 k8 ..) in the ready-made operand: hi terms; the lo terms lie 8 units further
static __host__ __device__ inline int few_unit(int m, int k8) { return (k8 >> 2) * 64 + (k8 & 3) * 16 + m; }
// out = X W^T (through RMSNorm if gain is given); out += X W^T; out = silu(gate) * up of norm(X); draft heads: rows
// [base + head][M] of h + silu(W_head h + bias), h = norm(X)
void launch_few_store(const FewLinear& a, hipStream_t s, hipEvent_t ev0 = nullptr, hipEvent_t ev1 = nullptr);
void launch_few_add(const FewLinear& a, hipStream_t s, hipEvent_t ev0 = nullptr, hipEvent_t ev1 = nullptr);
void launch_few_swiglu(const FewLinear& a, hipStream_t s, hipEvent_t ev0 = nullptr, hipEvent_t ev1 = nullptr);
void launch_few_heads(const FewLinear& a, const MedusaBias& bias, hipStream_t s, hipEvent_t ev0 = nullptr, hipEvent_t ev1 = nullptr);
// 9 to 32 rows, the contraction over the waves of a workgroup and S segments (gemm_kw.hip)
struct KwPlan { int C, S, RT; };                                      // column blocks of 16 (0: not that way), segments, tiles of 16 rows
KwPlan kw_plan(int M, int KB, int NB);
struct KwLinear {
    const void *X, *W;                                                // packed operands; KB * NB KiB < 4 GiB
    int KB, NB, M, S, n_units;                                        // n_units: columns / 16
    float* out; int ldo; size_t slot_stride;                          // partial sums [S][row][ldo]
};
void launch_gemm_kw(const KwPlan& p, const KwLinear& a, hipStream_t s, hipEvent_t ev0 = nullptr, hipEvent_t ev1 = nullptr);
// persistent layer kernel: G workgroups (all must be resident at once), a.MB in {1, 2, 8}
void launch_layer(const FusedArgs& a, int G, hipStream_t s, hipEvent_t ev0 = nullptr, hipEvent_t ev1 = nullptr);
// how many of its workgroups the device can hold at once (0 on error)
int fused_max_resident(int device);
// dst row i*B + b = summed row (i*M + sel[b]) - row0 of pv when it lies in [0, rows); i < H, b < B
void launch_reduce_selected(PartView pv, float* dst, const int32_t* sel, int B, int H, int M, int row0, int rows,
                            hipStream_t s);

// freq [head_dim / 2]: rotary frequencies
void launch_rope_freqs(double* freq, int hd, float theta, hipStream_t s);
void launch_build_rows_tree(RowTable rt, const int32_t* parent, const int32_t* depth, const int32_t* rank,
                            const int32_t* root_tok, const int32_t* cand, const int32_t* kv_len,
                            int B, int T, int Tp, int R, int H, int topk, int hd, const double* freq,
                            const void* embed, int embed_f32, int d, int V, float* x, hipStream_t s);
void launch_build_rows_chain(RowTable rt, const int32_t* tokens, const ChainArgs& ca, const RowMap& rm, PassMap* rm_dev, const int32_t* kv_len,
                             int B, int Tp, int hd, const double* freq, const void* embed, int embed_f32, int d, int V,
                             float* x, hipStream_t s);
// float32 device path (f32.hip): natural row-major layouts, float32 products
// out = norm(X[gather]) W^T (gain NULL: no norm); x += X W^T
void launch_f32_norm_linear(const float* X, const int32_t* gather, const float* gain, float eps, const float* W, float* out, int M,
                            int N, int K, int ldo, hipStream_t s);
void launch_f32_add_linear(const float* X, const float* W, float* x, int M, int N, int K, hipStream_t s);
// norm, QKV projection, rotary embedding: q [M][d], keys and values to the tree scratch
void launch_f32_qkv(const float* X, const float* gain, float eps, const float* W, RowTable rt, float* q, float* kt, float* vt, int M,
                    int nh, int hd, hipStream_t s);
void launch_f32_gate_up(const float* X, const float* gain, float eps, const float* W, float* act, int M, int F, int d,
                        hipStream_t s);
// out row i * B + b = h_b + silu(W_i h_b + bias_i), h_b = norm(X[gather[b]])
void launch_f32_heads(const float* X, const int32_t* gather, const float* gain, float eps, const float* W, const float* bias,
                      float* out, int B, int H, int d, hipStream_t s);
void launch_f32_attn(const float* q, const float* kc, const float* vc, const float* kt, const float* vt,
                     const int32_t* kv_len, const uint32_t* anc, float* out, RowRef rr, int longest, int B, int nh, int hd, int Tp,
                     int cap, hipStream_t s);
void launch_f32_kv_commit(const float* kt, const float* vt, float* kc, float* vc, const int32_t* src_slots,
                          const int32_t* n_accept, const int32_t* n_old, const RowMap& rm, const SeqList& row0, int kv_B, int L,
                          int B, int d, int rows, int cap, int W, hipStream_t s);
void launch_f32_kv_rows(float* kc, float* vc, float* k_rows, float* v_rows, int row0, int nrows, int d, int to_cache,
                        hipStream_t s);
void launch_norm_pack(float* x, PartView pv, const void* gain, float eps, void* xn_packed, float* hf_out,
                      int M, int d, int MB, const int32_t* gather, hipStream_t s);
void launch_rope_kv(PartView pv, RowTable rt, RowRef rr, void* q_packed, void* kt, void* vt, int B, int Tp, int nh,
                    int hd, hipStream_t s, const KvSinks* sinks = nullptr);
void launch_tree_attn(const void* q_packed, const void* kc, const void* vc, const void* kt, const void* vt,
                      const int32_t* kv_len, const uint32_t* anc, float* opart, float2* mlpart,
                      RowRef rr, int B, int nh, int hd, int Tp, int cap_blocks, int ncparts, int per, int tree_sep,
                      hipStream_t s, hipEvent_t ev0 = nullptr, hipEvent_t ev1 = nullptr, const PartView* qkv = nullptr,
                      const RowTable* rt = nullptr, const struct AttnSplit* split = nullptr);
// one workgroup per (sequence, head, 32 rows): the merged result, as a packed operand of MB row blocks. qkv, rt as above (Tp = 64)
void launch_attn_whole(const void* q_packed, const void* kc, const void* vc, void* kt, void* vt, const int32_t* kv_len,
                       const uint32_t* anc, void* x_packed, RowRef rr, int B, int nh, int hd, int Tp, int cap_blocks, int MB,
                       hipStream_t s, hipEvent_t ev0 = nullptr, hipEvent_t ev1 = nullptr, const PartView* qkv = nullptr,
                       const RowTable* rt = nullptr, int P = 1,
                       float* opart = nullptr, float2* mlpart = nullptr);
void launch_attn_merge(const float* opart, const float2* mlpart, void* x_packed, RowRef rr, int longest, int B, int nh, int hd,
                       int Tp, int nparts, int MB, hipStream_t s, const AttnSplit* split = nullptr);
// the same, as few.hip's ready-made operand
void launch_attn_merge_few(const float* opart, const float2* mlpart, void* out, RowRef rr, int longest, int B, int nh, int hd, int Tp,
                            int nparts, hipStream_t s, const AttnSplit* split = nullptr);
void launch_swiglu_pack(PartView pv, int F, int Fpad, void* act_packed, int M, int MB, hipStream_t s);
// output rows base * B + i*B + b in chunks of chunk_rows rows, each a packed activation of MB (last: MBlast) row blocks;
// base = 1: rows 0 .. B-1 are the h rows themselves
void launch_medusa_act(PartView pv, const float* h_rows, const MedusaBias& bias, int base, int B, int H, int d,
                       void* x_packed, int chunk_rows, int MB, int MBlast, hipStream_t s);
// Ranking of logit rows from partial sums (decide.hip); cand: device scratch of rows * rank_chunks(V) * k entries (k = 1 for
// launch_rank_best, whose result stays in it: per row and chunk {best logit, its id}); logits (or NULL): the summed rows
// are also written there, row r at logits + r * ld, and row (b, i) at head_logits + (b * H + i) * V
int rank_chunks(int V);
void launch_rank_best(PartView pv, int row0, int rows, int V, float* logits, int ld, float2* cand, hipStream_t s);
// out[seq[b]][i][0..k): ids of the largest k logits of row row0 + i * B + b, best first, lower id on ties
void launch_topk(PartView pv, int row0, int V, int k, int32_t* out, int B, int H, const SeqList& sl, float* head_logits,
                 void* cand, hipStream_t s);
// root_tok[seq[i]] = arg-max of ranked row i
void launch_pick_root(const float2* best, int V, int32_t* root_tok, int n, const SeqList& sl, hipStream_t s);
void launch_verify(const VerifyArgs& a, int B, hipStream_t s);
// per tree row: softmax statistics at a temperature and the typical-acceptance threshold (see decide.hip)
void launch_row_stats(const float* logits, int ld, int V, float4* stats, int B, int T, int Tp, float inv_temperature,
                      float epsilon, float delta, hipStream_t s);
// root_tok[b] = inverse-CDF draw at u[b] from softmax(logits[last_row[b]] * inv_temperature);
// -1 for a row index outside [0, n_rows)
void launch_sample_root(const float* logits, int ld, int V, const int32_t* last_row, const float* u,
                        float inv_temperature, int32_t* root_tok, int B, int n_rows, hipStream_t s);
// syntax-enriched label matrix [B][H+1][S] from the base label rows [B][S] (labels.hip)
void launch_build_labels(const int32_t* l0, int B, int S, int H, int32_t frag, int32_t pad, int32_t ignore,
                         int keep_all, int32_t* labels, hipStream_t s);
void launch_copy_row_stats(const float4* src, float4* dst, int B, int T, int Tp, hipStream_t s);
// commit: sequence i of the pass is sequence rm.seq[i] of the cache; rm.off[i] = its entry of the lists + 256 * its last row, to
// which slots are clamped (float32: counted from row row0.seq[i] of the scratch)
void launch_kv_commit(const void* kt_all, const void* vt_all, void* kc_all, void* vc_all,
                      const int32_t* src_slots, const int32_t* n_accept, const int32_t* n_old, const RowMap& rm, int kv_B,
                      int L, int B, int nh, int hd, int TB, int cap_blocks, int W, hipStream_t s);
// held: bit b set for every sequence that the tree scratch holds
void launch_commit_setup(const int32_t* n_rows, int width, uint32_t held, int B, int32_t* n_accept, int32_t* n_old,
                         int32_t* kv_len, hipStream_t s);
void launch_kv_rows(void* kc, void* vc, void* k_rows, void* v_rows, int row0, int nrows, int nh, int hd,
                    int cap_blocks, int to_cache, hipStream_t s);
void launch_fill_i32(int32_t* p, int32_t v, int n, hipStream_t s);
void launch_copy_i32(const int32_t* src, int32_t* dst, int n, const int32_t* src2, int32_t* dst2, int n2, hipStream_t s);
void launch_set_i32(const int32_t* v, int32_t* dst, int n, hipStream_t s);      // v: host, n <= SD_MAX_BATCH
void launch_prefill_commit_setup(const ChainArgs& ca, const RowMap& rm, int B, int Tp, int32_t* src_slots, int32_t* n_accept,
                                 int32_t* n_old, int32_t* kv_len, int32_t* fin_rows, int n_fin, const SeqList& last, hipStream_t s);
