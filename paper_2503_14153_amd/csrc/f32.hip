// The float32 device path: the same speculative step with weights, activations and the KV cache held as float32 and every
// product accumulated in float32. It exists for configurations that are specified in float32 (the small correctness
// configuration): shapes of that size are bound by the number of launches and by the latency of each, so the stages of a
// layer are five launches (projections carry the norm before them and the rotary embedding, the gate or the residual add
// after them), and a projection spreads its contraction over the eight waves of a workgroup, whose loads are all in
// flight together. Products run on the matrix cores in float32 (v_mfma_f32_16x16x4_f32: float32 operands, float32
// accumulation). The integer stages (tree assembly, ranking, acceptance, fragment cut) and the sampling statistics are the
// same kernels as on the bf16 path: they only ever see float32 logits.
// 16-node step of the small configuration (2 layers, d = 256): 470 us of kernels in 32 launches before, a projection of
// 32 x 256 outputs over 688 inputs 69 us (one 32 x 32 tile per workgroup, contraction blocks one after the other).
//
// Layouts: weights [out][in]; activations [row][col], rows packed as RowMap says; tree scratch [layer][row][d]; cache
// [layer][K|V][seq][cap][d].
#include "sd_internal.h"

// ------------------------------------------------------------------------------------------
// out = epilogue(norm(X) W^T). A workgroup of eight waves owns 32 rows x two blocks of 16 columns; wave w takes the
// contraction steps w, w + 8, .. of 16 and the waves' sums meet in LDS. Operands go from memory to the matrix cores: lane l
// loads four consecutive inputs of row (or column) l % 16, the four products of a step take one of them each, and since
// both operands are loaded alike, which input a product's contraction index stands for does not matter.
// NORM: X's rows go through RMSNorm: the operand is x * gain, the sums of squares ride along, and the row's 1 / rms factor
// is applied to the result (a product is linear in its rows).
// The two column blocks are chosen so that a thread of the epilogue holds what belongs together:
//   F32_STORE  columns 32t and 32t + 16: out[m][n] = v
//   F32_ADD    the same, added to out (the residual stream)
//   F32_QKV    dims i and i + hd/2 of one head: rotated at the row's position -> q; keys and values -> tree scratch
//   F32_GATE   gate column and up column: out[m][f] = silu(gate) * up
//   F32_HEADS  as STORE, z = v + bias[n]: out row (n / d) * M + m, column n % d: h + silu(z), h = the normalised row
enum { F32_STORE, F32_ADD, F32_QKV, F32_GATE, F32_HEADS };
struct F32Linear {
    const float *X, *gain, *W, *bias;
    const int32_t* gather;              // or NULL: row m reads X row gather[m]
    float eps;
    int M, N, K, ldo;
    float* out;
    float *kt, *vt;                     // F32_QKV
    const float2* cs;
    int nh, hd;
};
template <int MODE, bool NORM>
__global__ __launch_bounds__(512) void k_f32_linear(F32Linear a) {
    constexpr int NW = 8, U = 3;        // waves; steps whose loads are issued together
    __shared__ float red[NW][32][33];
    __shared__ float ssq[NW][32];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, r16 = lane & 15, kq = (lane >> 4) * 4;
    const int m0 = blockIdx.y * 32, t = blockIdx.x;
    int c0 = 32 * t, c1 = c0 + 16;
    if constexpr (MODE == F32_QKV) {
        const int per = a.hd / 32;      // 16-column blocks of a half head
        c0 = (t / per) * a.hd + (t % per) * 16;
        c1 = c0 + a.hd / 2;
    }
    if constexpr (MODE == F32_GATE) { c0 = 16 * t; c1 = a.N / 2 + 16 * t; }
    const float *xp[2], *wp[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {       // rows and columns past the end: the last one again, never stored
        const int m = min(m0 + 16 * i + r16, a.M - 1), n = min((i ? c1 : c0) + r16, a.N - 1);
        xp[i] = a.X + (size_t)(a.gather ? a.gather[m] : m) * a.K + kq;
        wp[i] = a.W + (size_t)n * a.K + kq;
    }
    f32x4 acc[2][2];
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[i >> 1][i & 1] = f32x4{0.f, 0.f, 0.f, 0.f};
    float ss[2] = {0.f, 0.f};
    const int S = a.K / 16;             // (d_model and d_ffn are multiples of 16)
    for (int s0 = wave; s0 < S; s0 += NW * U) {
        f32x4 x[U][2], w[U][2], g[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int s = min(s0 + NW * u, S - 1);
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                x[u][i] = *(const f32x4*)(xp[i] + 16 * s);
                w[u][i] = *(const f32x4*)(wp[i] + 16 * s);
            }
            if constexpr (NORM) g[u] = *(const f32x4*)(a.gain + 16 * s + kq);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (s0 + NW * u >= S) break;                   // wave-uniform
            if constexpr (NORM) {
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int e = 0; e < 4; ++e) { ss[i] = fmaf(x[u][i][e], x[u][i][e], ss[i]); x[u][i][e] *= g[u][e]; }
            }
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < 2; ++j)
                        acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(x[u][i][e], w[u][j][e], acc[i][j], 0, 0, 0);
        }
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) red[wave][16 * i + 4 * (lane >> 4) + v][16 * j + r16] = acc[i][j][v];
        if constexpr (NORM) {
            float q = ss[i];
            q += __shfl_xor(q, 16);
            q += __shfl_xor(q, 32);
            if (lane < 16) ssq[wave][16 * i + r16] = q;
        }
    }
    __syncthreads();
    const int row = tid >> 4, col = tid & 15, m = m0 + row;
    if (m >= a.M) return;
    float v0 = 0.f, v1 = 0.f, q = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        v0 += red[w][row][col];
        v1 += red[w][row][16 + col];
        if constexpr (NORM) q += ssq[w][row];
    }
    float r = 1.f;
    if constexpr (NORM) {
        r = rsqrtf(q / (float)a.K + a.eps);
        v0 *= r;
        v1 *= r;
    }
    const int n0 = c0 + col, n1 = c1 + col;
    if constexpr (MODE == F32_STORE || MODE == F32_ADD) {
        float* o = a.out + (size_t)m * a.ldo;
        if (n0 < a.N) o[n0] = MODE == F32_ADD ? o[n0] + v0 : v0;
        if (n1 < a.N) o[n1] = MODE == F32_ADD ? o[n1] + v1 : v1;
    } else if constexpr (MODE == F32_QKV) {
        const int d = a.nh * a.hd, which = n0 / d, c = n0 - which * d, i = c % a.hd;
        const size_t at = (size_t)m * d + c;
        float* o = which == 0 ? a.out : which == 1 ? a.kt : a.vt;
        if (which < 2) {
            const float2 cs = a.cs[(size_t)m * (a.hd / 2) + i];
            o[at] = v0 * cs.x - v1 * cs.y;
            o[at + a.hd / 2] = v1 * cs.x + v0 * cs.y;
        } else {
            o[at] = v0;
            o[at + a.hd / 2] = v1;
        }
    } else if constexpr (MODE == F32_GATE) {
        a.out[(size_t)m * a.ldo + n0] = v0 / (1.f + __expf(-v0)) * v1;
    } else {
        const float* xr = a.X + (size_t)(a.gather ? a.gather[m] : m) * a.K;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int n = i ? n1 : n0;
            if (n >= a.N) continue;
            const int head = n / a.K, c = n - head * a.K;
            const float z = (i ? v1 : v0) + a.bias[n];
            a.out[((size_t)head * a.M + m) * a.ldo + c] = xr[c] * r * a.gain[c] + z / (1.f + __expf(-z));
        }
    }
}

static void launch_linear(const F32Linear& a, int mode, bool norm, hipStream_t s) {
    const int tiles = mode == F32_GATE ? a.N / 32 : (a.N + 31) / 32;
    const dim3 grid(tiles, (a.M + 31) / 32), block(512);
    if (mode == F32_STORE && norm) hipLaunchKernelGGL((k_f32_linear<F32_STORE, true>), grid, block, 0, s, a);
    else if (mode == F32_STORE) hipLaunchKernelGGL((k_f32_linear<F32_STORE, false>), grid, block, 0, s, a);
    else if (mode == F32_ADD) hipLaunchKernelGGL((k_f32_linear<F32_ADD, false>), grid, block, 0, s, a);
    else if (mode == F32_QKV) hipLaunchKernelGGL((k_f32_linear<F32_QKV, true>), grid, block, 0, s, a);
    else if (mode == F32_GATE) hipLaunchKernelGGL((k_f32_linear<F32_GATE, true>), grid, block, 0, s, a);
    else hipLaunchKernelGGL((k_f32_linear<F32_HEADS, true>), grid, block, 0, s, a);
}
void launch_f32_norm_linear(const float* X, const int32_t* gather, const float* gain, float eps, const float* W, float* out, int M,
                            int N, int K, int ldo, hipStream_t s) {
    F32Linear a = {X, gain, W, nullptr, gather, eps, M, N, K, ldo, out, nullptr, nullptr, nullptr, 0, 0};
    launch_linear(a, F32_STORE, gain != nullptr, s);
}
void launch_f32_add_linear(const float* X, const float* W, float* x, int M, int N, int K, hipStream_t s) {
    F32Linear a = {X, nullptr, W, nullptr, nullptr, 0.f, M, N, K, N, x, nullptr, nullptr, nullptr, 0, 0};
    launch_linear(a, F32_ADD, false, s);
}
void launch_f32_qkv(const float* X, const float* gain, float eps, const float* W, RowTable rt, float* q, float* kt, float* vt, int M,
                    int nh, int hd, hipStream_t s) {
    const int d = nh * hd;
    F32Linear a = {X, gain, W, nullptr, nullptr, eps, M, 3 * d, d, d, q, kt, vt, rt.cs, nh, hd};
    launch_linear(a, F32_QKV, true, s);
}
void launch_f32_gate_up(const float* X, const float* gain, float eps, const float* W, float* act, int M, int F, int d,
                        hipStream_t s) {
    F32Linear a = {X, gain, W, nullptr, nullptr, eps, M, 2 * F, d, F, act, nullptr, nullptr, nullptr, 0, 0};
    launch_linear(a, F32_GATE, true, s);
}
void launch_f32_heads(const float* X, const int32_t* gather, const float* gain, float eps, const float* W, const float* bias,
                      float* out, int B, int H, int d, hipStream_t s) {
    F32Linear a = {X, gain, W, bias, gather, eps, B, H * d, d, d, out, nullptr, nullptr, nullptr, 0, 0};
    launch_linear(a, F32_HEADS, true, s);
}

// ------------------------------------------------------------------------------------------
// Tree-masked attention of one (sequence, head, row): softmax over the committed rows 0 .. n-1 and the tree rows in the
// row's ancestor set. The keys are dealt to the four waves in chunks of 64, one key per lane for the scores, one or two
// output dims per lane for the values, running maximum per wave; the waves merge through LDS.
template <int HD>
__global__ __launch_bounds__(256) void k_f32_attn(const float* __restrict__ q, const float* __restrict__ kc,
                                                  const float* __restrict__ vc, const float* __restrict__ kt,
                                                  const float* __restrict__ vt, const int32_t* __restrict__ kv_len,
                                                  const uint32_t* __restrict__ anc, float* __restrict__ out, RowRef rr, int nh,
                                                  int Tp, int cap, float scale) {
    constexpr int ND = HD / 64;         // output dims per lane
    const int t = blockIdx.x, h = blockIdx.y, b = blockIdx.z, d = nh * HD, tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int len = rr.len(b);
    if (t >= len) return;
    const int row0 = rr.off(b), m = row0 + t, sq = rr.seq(b), n = kv_len[sq], total = n + len;
    __shared__ __attribute__((aligned(16))) float qs[HD];
    __shared__ float mo[4][HD], ml[4][2];
    if (tid < HD) qs[tid] = q[(size_t)m * d + h * HD + tid];
    __syncthreads();
    const float* kcb = kc + (size_t)sq * cap * d + h * HD;
    const float* vcb = vc + (size_t)sq * cap * d + h * HD;
    const float* ktb = kt + (size_t)row0 * d + h * HD;
    const float* vtb = vt + (size_t)row0 * d + h * HD;
    const uint32_t* am = anc + ((size_t)b * Tp + t) * SD_ANC_WORDS;
    const float NINF = -__builtin_inff();
    float mrun = NINF, lrun = 0.f, o[ND];
#pragma unroll
    for (int e = 0; e < ND; ++e) o[e] = 0.f;
    for (int c0 = wave * 64; c0 < total; c0 += 256) {
        const int i = c0 + lane;
        bool vis = i < n;
        const float* kr = kcb + (size_t)min(i, max(n - 1, 0)) * d;
        if (i >= n) {
            const int j = min(i - n, len - 1);
            vis = i < total && ((am[j >> 5] >> (j & 31)) & 1u);
            kr = ktb + (size_t)j * d;
        }
        float s = 0.f;
#pragma unroll
        for (int e = 0; e < HD; e += 4) {
            const f32x4 k4 = *(const f32x4*)(kr + e), q4 = *(const f32x4*)(qs + e);
            s = fmaf(q4[0], k4[0], s); s = fmaf(q4[1], k4[1], s); s = fmaf(q4[2], k4[2], s); s = fmaf(q4[3], k4[3], s);
        }
        s = vis ? s * scale : NINF;
        float mx = s;
        for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
        const float mnew = fmaxf(mrun, mx);
        if (mnew == NINF) continue;                        // nothing visible so far (uniform over the wave)
        const float alpha = mrun == NINF ? 0.f : __expf(mrun - mnew);
        const float p = s == NINF ? 0.f : __expf(s - mnew);
        float ps = p;
        for (int off = 32; off > 0; off >>= 1) ps += __shfl_xor(ps, off);
        lrun = lrun * alpha + ps;
        mrun = mnew;
#pragma unroll
        for (int e = 0; e < ND; ++e) o[e] *= alpha;
        for (int j0 = 0; j0 < min(64, total - c0); j0 += 16) {
            float x[16][ND];                               // sixteen keys' values requested before the first is used
#pragma unroll
            for (int j = 0; j < 16; ++j) {                 // (past the end: the last key again, weight 0)
                const int k = min(c0 + j0 + j, total - 1);
                const float* vr = k < n ? vcb + (size_t)k * d : vtb + (size_t)(k - n) * d;
#pragma unroll
                for (int e = 0; e < ND; ++e) x[j][e] = vr[lane + 64 * e];
            }
#pragma unroll
            for (int j = 0; j < 16; ++j) {
                const float w = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(p), j0 + j));
#pragma unroll
                for (int e = 0; e < ND; ++e)               // (what is not visible never counts, not even as 0 x NaN)
                    o[e] = fmaf(w, w != 0.f ? x[j][e] : 0.f, o[e]);
            }
        }
    }
#pragma unroll
    for (int e = 0; e < ND; ++e) mo[wave][lane + 64 * e] = o[e];
    if (lane == 0) { ml[wave][0] = mrun; ml[wave][1] = lrun; }
    __syncthreads();
    if (tid < HD) {
        float M = NINF, L = 0.f, v = 0.f;
#pragma unroll
        for (int w = 0; w < 4; ++w) M = fmaxf(M, ml[w][0]);
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            const float f = ml[w][0] == NINF ? 0.f : __expf(ml[w][0] - M);
            L += f * ml[w][1];
            v += f * mo[w][tid];
        }
        out[(size_t)m * d + h * HD + tid] = L > 0.f ? v / L : 0.f;
    }
}
void launch_f32_attn(const float* q, const float* kc, const float* vc, const float* kt, const float* vt,
                     const int32_t* kv_len, const uint32_t* anc, float* out, RowRef rr, int longest, int B, int nh, int hd, int Tp,
                     int cap, hipStream_t s) {
    const dim3 grid(longest, nh, B);
    const float scale = 1.f / sqrtf((float)hd);
    if (hd == 128)
        hipLaunchKernelGGL(k_f32_attn<128>, grid, dim3(256), 0, s, q, kc, vc, kt, vt, kv_len, anc, out, rr, nh, Tp, cap, scale);
    else
        hipLaunchKernelGGL(k_f32_attn<64>, grid, dim3(256), 0, s, q, kc, vc, kt, vt, kv_len, anc, out, rr, nh, Tp, cap, scale);
}

// ------------------------------------------------------------------------------------------
// Commit: row src_slots[list][j] of pass sequence i -> cache row n_old[list] + j of sequence rm.seq[i], for j < n_accept[list],
// every layer, K and V; rm.off[i] = list + 256 * the sequence's last row. Its rows start at scratch row row0.seq[i]; a slot past
// the last gives the last, never another sequence's row. grid (row j, layer * B + i), 64 threads over the d columns.
__global__ void k_f32_kv_commit(const float* __restrict__ kt, const float* __restrict__ vt, float* __restrict__ kc,
                                float* __restrict__ vc, const int32_t* __restrict__ src_slots,
                                const int32_t* __restrict__ n_accept, const int32_t* __restrict__ n_old, RowMap rm, SeqList row0,
                                int B, int d, int cap, int W, size_t layer_stride_t, size_t layer_stride_c) {
    const int j = blockIdx.x, l = blockIdx.y / B, i = blockIdx.y % B, lst = rm.off[i] & 255;
    if (j >= min(n_accept[lst], W)) return;
    const int src = row0.seq[i] + min(max(src_slots[(size_t)lst * W + j], 0), rm.off[i] >> 8), dst = n_old[lst] + j;
    const size_t so = l * layer_stride_t + (size_t)src * d, dofs = l * layer_stride_c + ((size_t)rm.seq[i] * cap + dst) * d;
    for (int c = threadIdx.x * 4; c < d; c += blockDim.x * 4) {
        *(f32x4*)(kc + dofs + c) = *(const f32x4*)(kt + so + c);
        *(f32x4*)(vc + dofs + c) = *(const f32x4*)(vt + so + c);
    }
}
void launch_f32_kv_commit(const float* kt, const float* vt, float* kc, float* vc, const int32_t* src_slots,
                          const int32_t* n_accept, const int32_t* n_old, const RowMap& rm, const SeqList& row0, int kv_B, int L,
                          int B, int d, int rows, int cap, int W, hipStream_t s) {
    hipLaunchKernelGGL(k_f32_kv_commit, dim3(W, L * B), dim3(64), 0, s, kt, vt, kc, vc, src_slots, n_accept, n_old, rm, row0, B, d,
                       cap, W, (size_t)rows * d, (size_t)kv_B * cap * d);
}

// natural-layout rows [nrows][d] <-> cache rows of one sequence and layer
__global__ void k_f32_kv_rows(float* __restrict__ kc, float* __restrict__ vc, float* __restrict__ k_rows,
                              float* __restrict__ v_rows, int row0, int d, int to_cache) {
    const int r = blockIdx.x;
    for (int c = threadIdx.x; c < d; c += blockDim.x) {
        const size_t ci = (size_t)(row0 + r) * d + c, ni = (size_t)r * d + c;
        if (to_cache) { kc[ci] = k_rows[ni]; vc[ci] = v_rows[ni]; }
        else { k_rows[ni] = kc[ci]; v_rows[ni] = vc[ci]; }
    }
}
void launch_f32_kv_rows(float* kc, float* vc, float* k_rows, float* v_rows, int row0, int nrows, int d, int to_cache,
                        hipStream_t s) {
    hipLaunchKernelGGL(k_f32_kv_rows, dim3(nrows), dim3(256), 0, s, kc, vc, k_rows, v_rows, row0, d, to_cache);
}
