// Projections of 9 to 32 rows whose contraction is dealt to the WAVES of a workgroup ("kw"). k_gemm_sk gives every wave a
// column block of its own and shares the activations through LDS: few activation bytes, but every workgroup leaves a whole
// 256-column tile of partial sums, and filling the chip takes 4 to 16 of those per column. Here a workgroup has C blocks of 16
// columns, its eight waves take the steps of the contraction (32 inputs) in turn, each with its own operands straight from
// memory, and their sums meet in LDS: S partial tiles per column instead, at most eight (7B shape 1 to 4, 13B 1 to 5, more at small widths).
// Bound by what the L2s deliver (10.6 TB/s): a workgroup reads 32 C bytes of weights and 4 M of activations per input. At 32 rows
// that is below the weight stream's own time; at 64 rows the activations are most of the bytes and k_gemm_sk is as fast or
// faster. 7B shape, launches on their own, k_gemm_sk -> here, us (slots): 32 rows QKV 22.1 -> 18.7 (4 -> 2), O 10.1 -> 8.4
// (8 -> 4), down 17.5 -> 16.8 (16 -> 4). Steps of four layers, one sequence: 16 nodes 662 -> 618, 32 nodes 669 -> 642; 13B
// shape, 12 nodes 832 -> 786, 30 nodes 868 -> 846. Not kept: 64 rows (QKV level at the 7B shape, 13B step 962 -> 982; O and down
// slower), and gate/up with SwiGLU in the epilogue (32 rows 680 -> 714).
#include "sd_internal.h"
#include "row_ops.h"

// RT tiles of 16 rows; the operand is a packed activation of one row block (sd_internal.h): half a fragment of two contraction
// blocks that lie one above the other is the 16 x 32 operand of the product, and so it is with the weights.
template <int RT, int C, int R>
__global__ __launch_bounds__(512, 2) void k_gemm_kw(KwLinear a) {
    constexpr int NW = 8;
    __shared__ float red[2][NW][C][16 * 17];
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, c16 = lane & 15, kg = lane >> 4;
    const int g = blockIdx.x / a.S, seg = blockIdx.x - g * a.S;
    const int steps = (a.KB + 1) >> 1, s0 = steps * seg / a.S, s1 = steps * (seg + 1) / a.S;      // S <= steps
    const int mine = s1 - s0 > wave ? (s1 - s0 - wave + NW - 1) / NW : 0, groups = (mine + R - 1) / R;
    const char *Wb = (const char*)a.W, *Xb = (const char*)a.X;
    uint32_t wo[C];                                    // byte offsets (32 bits: a matrix is smaller than 4 GiB)
#pragma unroll
    for (int c = 0; c < C; ++c) {
        const int hb = min(g * C + c, a.n_units - 1);
        wo[c] = (uint32_t)(((hb >> 1) * 64 + (hb & 1) * 16 + c16 + 32 * (kg & 1)) * 16);
    }
    const uint32_t kb_bytes = (uint32_t)a.NB * 1024u, xo = (uint32_t)((c16 + 32 * (kg & 1)) * 16);
    bf16x8 w[R][C], x[R][RT][2];
    auto load = [&](int j, int i) {                    // step `i` of this wave -> ring slot j; past the end the last step again
        const int s = min(s0 + wave + NW * i, s1 - 1);
        const uint32_t kb = (uint32_t)min(2 * s + (kg >> 1), a.KB - 1), xa = kb * 2048u + xo, at = kb * kb_bytes;
#pragma unroll
        for (int t = 0; t < RT; ++t)
#pragma unroll
            for (int p = 0; p < 2; ++p)
                x[j][t][p] = *(const bf16x8*)(Xb + (xa + (uint32_t)(p * 1024 + t * 256)));
#pragma unroll
        for (int c = 0; c < C; ++c) w[j][c] = __builtin_nontemporal_load((const bf16x8*)(Wb + (at + wo[c])));
    };
#pragma unroll
    for (int j = 0; j < R; ++j) load(j, j);
    f32x4 acc[C][RT];
#pragma unroll
    for (int c = 0; c < C; ++c)
#pragma unroll
        for (int t = 0; t < RT; ++t) acc[c][t] = f32x4{0.f, 0.f, 0.f, 0.f};
    auto multiply = [&](int j, int i, bool last) {
        if (last) {                                    // (compile-time: the last group is a copy of its own) zeros past the end,
            const int s = s0 + wave + NW * i;          // in both operands: what lies there need not be finite
            const bool ok = s < s1 && s * 32 + kg * 8 < a.KB * 16;
            auto keep = [&](bf16x8& v) {
                union { bf16x8 b; uint4 u; } o = {v};
                o.u = make_uint4(ok ? o.u.x : 0u, ok ? o.u.y : 0u, ok ? o.u.z : 0u, ok ? o.u.w : 0u);
                v = o.b;
            };
#pragma unroll
            for (int c = 0; c < C; ++c) keep(w[j][c]);
#pragma unroll
            for (int t = 0; t < RT; ++t) { keep(x[j][t][0]); keep(x[j][t][1]); }
        }
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
            for (int t = 0; t < RT; ++t)
#pragma unroll
                for (int c = 0; c < C; ++c) acc[c][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(x[j][t][p], w[j][c], acc[c][t], 0, 0, 0);
    };
    for (int q = 0; q + 1 < groups; ++q) {
#pragma unroll
        for (int j = 0; j < R; ++j) {
            multiply(j, q * R + j, false);
            load(j, (q + 1) * R + j);
        }
    }
    if (groups > 0) {
#pragma unroll
        for (int j = 0; j < R; ++j) multiply(j, (groups - 1) * R + j, true);
    }
    // The waves' sums, 16 rows at a time through two buffers (whoever writes a buffer again has passed the barrier after the
    // one that its readers had passed). A lane holds column c16, rows 4 kg .. 4 kg + 3.
#pragma unroll
    for (int t = 0; t < RT; ++t) {
        float(*rd)[C][16 * 17] = red[t & 1];
#pragma unroll
        for (int c = 0; c < C; ++c)
#pragma unroll
            for (int v = 0; v < 4; ++v) rd[wave][c][(4 * kg + v) * 17 + c16] = acc[c][t][v];
        __syncthreads();
        for (int i = tid; i < 16 * C * 4; i += NW * 64) {  // four columns of a row
            const int q = i & 3, c = (i >> 2) % C, r = (i >> 2) / C, m = t * 16 + r, unit = g * C + c;
            if (m >= a.M || unit >= a.n_units) continue;
            float f[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                f[e] = 0.f;
#pragma unroll
                for (int p = 0; p < NW; ++p) f[e] += rd[p][c][r * 17 + q * 4 + e];
            }
            *(float4*)(a.out + (size_t)seg * a.slot_stride + (size_t)m * a.ldo + unit * 16 + q * 4) = make_float4(f[0], f[1], f[2], f[3]);
        }
    }
}

// Column blocks and segments: the time of a workgroup at the rate that one compute unit gets from L2 (45 KB per us), the weight
// stream (6 TB/s), and the partial tiles, written and read again at 4.5 TB/s.
KwPlan kw_plan(int M, int KB, int NB) {
    static const int widths[] = {2, 3, 4, 6, 8};
    const int RT = M <= 16 ? 1 : 2, units = NB * 2, steps = (KB + 1) / 2;
    KwPlan p = {0, 0, RT};
    double best = 0;
    for (int C : widths) {
        const int groups = (units + C - 1) / C;
        for (int S = 1; S <= 8 && S <= steps; ++S) {
            const int rounds = (groups * S + 255) / 256;
            const double wg = (double)((steps + S - 1) / S) * (C + 2 * RT) * 1024 / 45000, stream = (double)KB * NB * 1024 / 6e6;
            const double cost = (rounds * wg > stream ? rounds * wg : stream) + (double)S * M * NB * 32 * 8 / 4.5e6;
            if (p.C == 0 || cost < best) { best = cost; p.C = C; p.S = S; }
        }
    }
    return p;
}

void launch_gemm_kw(const KwPlan& p, const KwLinear& a, hipStream_t s, hipEvent_t ev0, hipEvent_t ev1) {
    const int grid = (a.n_units + p.C - 1) / p.C * p.S;
#define KW_GO(RT_, C_)                                                                                                   \
    do {                                                                                                                 \
        constexpr int R_ = RT_ == 1 ? 2 : 1;                                                                             \
        if (ev0 || ev1) hipExtLaunchKernelGGL((k_gemm_kw<RT_, C_, R_>), dim3(grid), dim3(512), 0, s, ev0, ev1, 0, a);    \
        else hipLaunchKernelGGL((k_gemm_kw<RT_, C_, R_>), dim3(grid), dim3(512), 0, s, a);                               \
    } while (0)
#define KW_RT(C_) do { if (p.RT == 1) KW_GO(1, C_); else KW_GO(2, C_); } while (0)
    if (p.C == 2) KW_RT(2); else if (p.C == 3) KW_RT(3); else if (p.C == 4) KW_RT(4); else if (p.C == 6) KW_RT(6); else KW_RT(8);
#undef KW_RT
#undef KW_GO
}
