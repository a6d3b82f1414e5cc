// Projections of a handful of rows (plain decoding, small trees, the draft heads): out = epilogue(source(X) W^T) with every
// output column finished by ONE workgroup. With 64 rows a column block's share of the contraction is cut over workgroups and
// the row-wise kernels in between sum the partial tiles; with up to 16 rows the activations are so small that a workgroup can
// read all of them, so nothing is cut: the eight waves of a workgroup take the steps of the contraction in turn, their sums
// meet in LDS, and norm, residual add, SwiGLU and the draft heads' activation happen where the operand is made and where the
// sums are. A layer is five launches (six beyond two rows: the merge of the attention parts) instead of nine.
//
// Bound by the weight stream. A workgroup owns C blocks of 16 columns, a step is 32 inputs of them: C products of 16 x 16 x 32.
// The weights' 1 KiB fragments hold 32 columns x 16 inputs; half a column block of two fragments that lie one above the
// other is the 16 x 32 operand, four runs of 256 contiguous bytes. Every wave keeps R steps in flight.
// The activations enter as two bfloat16 terms (hi + lo) like everywhere else. Up to eight rows both terms ride in ONE product:
// rows 0-7 of the operand are the hi terms, rows 8-15 the lo terms, added at the end. Up to 16 rows take two products.
// Where a workgroup has one column block (O and down projection) making the operand from float32 rows is more work than a
// step's weights take to arrive, so there it comes ready-made: [step][lane][8], 1 KiB a step (sd_internal.h few_unit),
// written by the attention merge (or here, into LDS) and by the SwiGLU epilogue.
#include "sd_internal.h"
#include "row_ops.h"

enum { FEW_STORE, FEW_ADD, FEW_SWIGLU, FEW_HEADS };   // what becomes of the sums
enum { FEW_ROWS_AS_THEY_ARE, FEW_NORM, FEW_PACKED, FEW_MERGE };   // where the operand comes from

template <int MODE, int SRC, int C, int R, int MR>
static __device__ __forceinline__ void few_body(const FewLinear& a, const MedusaBias* bias, bf16x8* merged) {
    constexpr int U = MODE == FEW_SWIGLU ? C / 2 : C;  // units of a workgroup: column blocks, or pairs (gate block, up block)
    constexpr int NW = 8;                              // waves
    constexpr int NX = MR / 8;                         // products per step and column block
    constexpr bool READY = SRC == FEW_PACKED || SRC == FEW_MERGE;
    static_assert(!READY || MR == 8, "one product a step");
    __shared__ float red[NW][C][16 * 17];
    __shared__ float ssq[NW][16];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, c16 = lane & 15, kg = lane >> 4;
    const int K = a.KB * 16, S = (a.KB + 1) >> 1;      // steps; the last one may be half (lanes past the end: zero operand)
    const int mine = S > wave ? (S - wave + NW - 1) / NW : 0, groups = (mine + R - 1) / R;

    // weights: byte offset of this lane in column block c (32 bits: a matrix is smaller than 4 GiB)
    const char* Wb = (const char*)a.W;
    uint32_t wo[C];
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const int hb = min((int)blockIdx.x * U + c % U, a.n_units - 1) + (c >= U ? a.up : 0);
        wo[c] = (uint32_t)(((hb >> 1) * 64 + (hb & 1) * 16 + c16 + 32 * (kg & 1)) * 16);
    }
    const uint32_t kb_bytes = (uint32_t)a.NB * 1024u;
    const int row = min(lane & (MR - 1), a.M - 1);
    const int ready_at = kg * 16 + (c16 & 8) + row;    // this lane's piece of a step of the ready-made operand
    const float* xr = READY ? nullptr : a.X + (size_t)(a.gather ? a.gather[row] : row) * a.ldx;
    bf16x8 w[R][C], xp[R];
    f32x4 x[R][2];
    uint4 gn[R];
    auto load = [&](int j, int i) {                    // step `i` of this wave -> ring slot j; past the end the last step again
        const int s = min(wave + NW * i, S - 1), k = min(s * 32 + kg * 8, K - 8);
        if constexpr (SRC == FEW_PACKED) xp[j] = a.Xp[(size_t)s * 64 + ready_at];
        if constexpr (!READY) {
            x[j][0] = *(const f32x4*)(xr + k);
            x[j][1] = *(const f32x4*)(xr + k + 4);
        }
        if constexpr (SRC == FEW_NORM) gn[j] = *(const uint4*)(a.gain + k);
        const uint32_t at = (uint32_t)min(2 * s + (kg >> 1), a.KB - 1) * kb_bytes;
#pragma unroll
        for (int c = 0; c < C; ++c) w[j][c] = __builtin_nontemporal_load((const bf16x8*)(Wb + (at + wo[c])));
    };
#pragma unroll
    for (int j = 0; j < R; ++j) load(j, j);
    if constexpr (SRC == FEW_MERGE) {                  // merged attention output of all rows -> LDS, while the first weights arrive
        const int e8s = a.hd == 128 ? 4 : 3, per = K >> 3;
        for (int i = tid; i < a.M * per; i += NW * 64) {
            const int m = i / per, k8 = i - m * per, b = m / a.R;
            float f[8];
            attn_merge_values(a.opart, a.mlpart, a.nh, a.hd, a.Tp, a.nparts, b ? a.own[1] : a.own[0], b, k8 >> e8s, m - b * a.R, k8 & ((1 << e8s) - 1), f);
            bf16x8 hi, lo;
            split_hilo(f, hi, lo);
            merged[k8 * (2 * FEW_MERGE_ROWS) + m] = hi;
            merged[k8 * (2 * FEW_MERGE_ROWS) + FEW_MERGE_ROWS + m] = lo;
        }
        __syncthreads();
    }
    f32x4 acc[C];
#pragma unroll
    for (int c = 0; c < C; ++c) acc[c] = f32x4{0.f, 0.f, 0.f, 0.f};
    float ss = 0.f;
    auto multiply = [&](int j, int i, bool last) {
        const int s = wave + NW * i;                        // (last: compile-time, the last group is a copy of its own)
        const bool ok = !last || (s < S && s * 32 + kg * 8 < K);
        if constexpr (READY) {
            union { bf16x8 b; uint4 u; } o;
            if constexpr (SRC == FEW_MERGE)
                o.b = merged[min(min(s, S - 1) * 4 + kg, 2 * a.KB - 1) * (2 * FEW_MERGE_ROWS) + (c16 >> 3) * FEW_MERGE_ROWS + row];
            else o.b = xp[j];
            if (last) o.u = make_uint4(ok ? o.u.x : 0u, ok ? o.u.y : 0u, ok ? o.u.z : 0u, ok ? o.u.w : 0u);
#pragma unroll
            for (int c = 0; c < C; ++c) acc[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(o.b, w[j][c], acc[c], 0, 0, 0);
            return;
        }
        float f[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) f[e] = x[j][e >> 2][e & 3];
        if (last)
#pragma unroll
            for (int e = 0; e < 8; ++e) f[e] = ok ? f[e] : 0.f;
        if constexpr (SRC == FEW_NORM) {
            const uint32_t g[4] = {gn[j].x, gn[j].y, gn[j].z, gn[j].w};
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                ss = fmaf(f[e], f[e], ss);
                f[e] *= __uint_as_float((e & 1) ? (g[e >> 1] & 0xffff0000u) : (g[e >> 1] << 16));
            }
        }
        bf16x8 hi, lo;
        split_hilo(f, hi, lo);
        if constexpr (MR == 8) {
            const bool up = (lane & 8) != 0;
            union { bf16x8 b; uint4 u; } h = {hi}, l = {lo}, o;
            o.u = make_uint4(up ? l.u.x : h.u.x, up ? l.u.y : h.u.y, up ? l.u.z : h.u.z, up ? l.u.w : h.u.w);
#pragma unroll
            for (int c = 0; c < C; ++c) acc[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(o.b, w[j][c], acc[c], 0, 0, 0);
        } else {
#pragma unroll
            for (int c = 0; c < C; ++c) acc[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(hi, w[j][c], acc[c], 0, 0, 0);
#pragma unroll
            for (int c = 0; c < C; ++c) acc[c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(lo, w[j][c], acc[c], 0, 0, 0);
        }
    };
    for (int g = 0; g + 1 < groups; ++g) {
#pragma unroll
        for (int j = 0; j < R; ++j) {
            multiply(j, g * R + j, false);
            load(j, (g + 1) * R + j);
        }
    }
    if (groups > 0) {
#pragma unroll
        for (int j = 0; j < R; ++j) multiply(j, (groups - 1) * R + j, true);
    }
    // the waves' sums: lane holds column c16, rows 4 kg .. 4 kg + 3
#pragma unroll
    for (int c = 0; c < C; ++c)
#pragma unroll
        for (int v = 0; v < 4; ++v) red[wave][c][(4 * kg + v) * 17 + c16] = acc[c][v];
    if constexpr (SRC == FEW_NORM) {
        ss += __shfl_xor(ss, 16);
        ss += __shfl_xor(ss, 32);
        if (lane < 16) ssq[wave][lane] = ss;
    }
    __syncthreads();
    auto sum = [&](int c, int m, int col) {
        float t = 0.f;
#pragma unroll
        for (int p = 0; p < NW; ++p) t += red[p][c][m * 17 + col];
        if constexpr (NX == 1)
#pragma unroll
            for (int p = 0; p < NW; ++p) t += red[p][c][(m + 8) * 17 + col];
        return t;
    };
    for (int i = tid; i < a.M * U * 16; i += NW * 64) {
        const int col = i & 15, u = (i >> 4) % U, m = (i >> 4) / U, unit = blockIdx.x * U + u;
        if (unit >= a.n_units) continue;
        float r = 1.f;
        if constexpr (SRC == FEW_NORM) {
            float q = 0.f;
#pragma unroll
            for (int p = 0; p < NW; ++p) q += ssq[p][m];
            r = rsqrtf(q / (float)K + a.eps);
        }
        if constexpr (SRC == FEW_ROWS_AS_THEY_ARE)
            if (a.row_scale) r = a.row_scale[m];
        const float v = sum(u, m, col) * r;
        const int n = unit * 16 + col;
        if constexpr (MODE == FEW_STORE) {
            a.out[(size_t)m * a.ldo + n] = v;
        } else if constexpr (MODE == FEW_ADD) {
            a.out[(size_t)m * a.ldo + n] += v;
        } else if constexpr (MODE == FEW_SWIGLU) {
            const float up = sum(U + u, m, col) * r;
            const float y = v / (1.f + __expf(-v)) * up;
            const __bf16 hi = (__bf16)y;
            __bf16* d = (__bf16*)a.packed + (size_t)few_unit(m, n >> 3) * 8 + (n & 7);
            d[0] = hi;
            d[64] = (__bf16)(y - (float)hi);
        } else {                                       // draft head n / K: h + silu(v + bias), h the normalised row
            const int head = n / K, c = n - head * K, at = (head + a.base) * a.M + m;
            const float xg = a.X[(size_t)(a.gather ? a.gather[m] : m) * a.ldx + c] * bf16_bits_to_float(a.gain[c]), h = xg * r;
            const uint16_t* bi = bias->p[head];
            const float z = v + (bi ? bf16_bits_to_float(bi[c]) : 0.f);
            const float y = h + z / (1.f + __expf(-z));
            if (a.packed) {                            // more rows than this path's LM head takes: the wide one's operand
                const auto put = [&](int at_, float f) {
                    const __bf16 hi = (__bf16)f;
                    __bf16* d = (__bf16*)a.packed + xpack_index(at_, c, a.MB);
                    d[0] = hi;
                    d[XPART] = (__bf16)(f - (float)hi);
                };
                put(at, y);
                if (a.base && head == 0) put(m, h);
                continue;
            }
            a.out[(size_t)at * a.ldo + c] = y;
            if (c == 0) a.scale_out[at] = 1.f;
            if (a.base && head == 0) {                 // the base rows in front of the heads'
                a.out[(size_t)m * a.ldo + c] = xg;
                if (c == 0) a.scale_out[m] = r;
            }
        }
    }
}

template <int MODE, int SRC, int C, int R, int MR>
__global__ __launch_bounds__(512, C <= 2 && SRC != FEW_MERGE && SRC != FEW_NORM ? 4 : 2) void k_few(FewLinear a) {
    extern __shared__ bf16x8 merged[];
    few_body<MODE, SRC, C, R, MR>(a, nullptr, merged);
}
template <int C, int R, int MR>
__global__ __launch_bounds__(512, 2) void k_few_heads(FewLinear a, MedusaBias bias) {
    few_body<FEW_HEADS, FEW_NORM, C, R, MR>(a, &bias, nullptr);
}

// Column blocks per workgroup: as few as keep the grid at `most` workgroups (256: one per compute unit; 512 where two share
// one). R: four to sixteen fragments in flight per wave. 7B shape, one row, us: QKV 3 blocks on 256 workgroups 18.3, 2 on 384
// 20.6; down projection (43 steps a wave) R = 4 / 8 / 11: 17.6 / 18.6 / 18.2, with 16 waves 18.4, 2 blocks on 128 24.
// What it replaced (k_gemm_sk and the row-wise launches between): per layer norm 5.2 + QKV 21.2 + attention 10.9 + O 10.4 +
// norm 5.2 + gate/up 31.2 + down 18.2; now 18.3 + 10.8 + 9.8 + 28.4 + 17.6. Plain decoding of four layers 592 -> 516 us,
// of eight sequences 907 -> 809. Beyond eight rows an operand of two products a step is as many bytes as the weights.
static int few_width(int units, const int* widths, int n, int most) {
    for (int i = 0; i < n; ++i)
        if ((units + widths[i] - 1) / widths[i] <= most) return widths[i];
    return widths[n - 1];
}

#define FEW_GO(KERNEL_, LDS_, ...)                                                                         \
    do {                                                                                                   \
        if (ev0 || ev1) hipExtLaunchKernelGGL(KERNEL_, dim3(grid), dim3(512), LDS_, s, ev0, ev1, 0, __VA_ARGS__); \
        else hipLaunchKernelGGL(KERNEL_, dim3(grid), dim3(512), LDS_, s, __VA_ARGS__);                     \
    } while (0)
#define FEW_MR(MODE_, SRC_, C_, R_, LDS_)                                                                  \
    do { if (a.M <= 8) FEW_GO((k_few<MODE_, SRC_, C_, R_, 8>), LDS_, a); else FEW_GO((k_few<MODE_, SRC_, C_, R_, 16>), LDS_, a); } while (0)

void launch_few_store(const FewLinear& a, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
    static const int widths[] = {2, 3, 4, 6, 8};
    const int C = few_width(a.n_units, widths, 5, 256), grid = (a.n_units + C - 1) / C;
#define FEW_STORE_C(SRC_)                                                                                  \
    switch (C) {                                                                                           \
    case 2: FEW_MR(FEW_STORE, SRC_, 2, 4, 0); break;                                                       \
    case 3: FEW_MR(FEW_STORE, SRC_, 3, 4, 0); break;                                                       \
    case 4: FEW_MR(FEW_STORE, SRC_, 4, 3, 0); break;                                                       \
    case 6: FEW_MR(FEW_STORE, SRC_, 6, 2, 0); break;                                                       \
    default: FEW_MR(FEW_STORE, SRC_, 8, 2, 0); break;                                                      \
    }
    if (a.gain) FEW_STORE_C(FEW_NORM) else FEW_STORE_C(FEW_ROWS_AS_THEY_ARE)
#undef FEW_STORE_C
}
void launch_few_add(const FewLinear& a, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
    static const int widths[] = {1, 2};
    const int C = few_width(a.n_units, widths, 2, a.opart ? 256 : 512), grid = (a.n_units + C - 1) / C;
    const size_t lds = (size_t)a.KB * 2 * (2 * FEW_MERGE_ROWS) * 16;
    if (a.opart) {
        if (C == 1) FEW_GO((k_few<FEW_ADD, FEW_MERGE, 1, 8, 8>), lds, a); else FEW_GO((k_few<FEW_ADD, FEW_MERGE, 2, 4, 8>), lds, a);
    } else {
        if (C == 1) FEW_GO((k_few<FEW_ADD, FEW_PACKED, 1, 4, 8>), 0, a); else FEW_GO((k_few<FEW_ADD, FEW_PACKED, 2, 4, 8>), 0, a);
    }
}
void launch_few_swiglu(const FewLinear& a, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
    static const int widths[] = {1, 2, 3, 4};          // pairs
    const int P = few_width(a.n_units, widths, 4, 256), grid = (a.n_units + P - 1) / P;
    switch (P) {
    case 1: FEW_GO((k_few<FEW_SWIGLU, FEW_NORM, 2, 4, 8>), 0, a); break;
    case 2: FEW_GO((k_few<FEW_SWIGLU, FEW_NORM, 4, 3, 8>), 0, a); break;
    case 3: FEW_GO((k_few<FEW_SWIGLU, FEW_NORM, 6, 2, 8>), 0, a); break;
    default: FEW_GO((k_few<FEW_SWIGLU, FEW_NORM, 8, 2, 8>), 0, a); break;
    }
}
void launch_few_heads(const FewLinear& a, const MedusaBias& bias, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
    static const int widths[] = {2, 4, 6, 8};
    const int C = few_width(a.n_units, widths, 4, 256), grid = (a.n_units + C - 1) / C;
#define FEW_HEADS_C(C_, R_)                                                                                \
    do { if (a.M <= 8) FEW_GO((k_few_heads<C_, R_, 8>), 0, a, bias); else FEW_GO((k_few_heads<C_, R_, 16>), 0, a, bias); } while (0)
    switch (C) {
    case 2: FEW_HEADS_C(2, 4); break;
    case 4: FEW_HEADS_C(4, 3); break;
    case 6: FEW_HEADS_C(6, 2); break;
    default: FEW_HEADS_C(8, 2); break;
    }
#undef FEW_HEADS_C
}
