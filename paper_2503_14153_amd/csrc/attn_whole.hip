// Tree-masked attention with ONE workgroup per (sequence, head, 32 query rows): its eight waves share the sequence's blocks, meet
// in LDS and write the merged, normalised result as the next projection's operand. No parts, no partials in memory, no merge
// launch, and rows past the first block no longer ride with 64 others. attn.hip cuts a head's blocks over several workgroups
// instead, which a long sequence needs: a workgroup takes about 0.16 us per block and 32 rows (32 MFMAs on two-term queries and
// probabilities, the softmax and 16 KiB of queries from LDS each), so this one is for few blocks (attn_whole_parts).
// 7B shape, steps of four layers, us, parts and merge -> here: 64 nodes over 300 rows 700 -> 680, over 700 716 -> 711, over 1800 735
// -> 750; 128 nodes over 1000 942 -> 926; 256 over 512 1302 -> 1264; two sequences of 500 and 900, 64 nodes 939 -> 914; 13B
// shape, 128 over 4096 1267 -> 1287; one row block never (plain decoding over 1000 rows 441 -> 471). Holding two blocks of
// keys instead of one changes nothing.
//
// PARTS: a workgroup takes one of P equal shares of the blocks (the last one the tree's too) and leaves partial results as attn.hip
// does, for the same merge: attn_whole_parts has where and what it gives.
//
// Arithmetic, layouts and masks as in attn.hip (S^T = K Q^T, values permuted so that exp(S) is the next operand, two-term queries
// and probabilities, lazily raised maximum). A wave holds one block of keys and values and asks for the next as soon as the
// registers are free; two waves per SIMD (at most 256 registers each) cover one another's waits and softmax.
//
// FR: no rotary launch before this one: the workgroup builds its queries from the QKV projection's partial sums, and the tree's
// keys and values of the blocks its rows can see, in LDS; block tg also goes to the scratch, for the commit.
#include "sd_internal.h"
#include "row_ops.h"

typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
#define NEG_INF (-__builtin_inff())
#define LAZY_MAX 8.0f                  // the running maximum is raised only past 2^8 of itself (see attn.hip)

template <int HD, int AW, int FR, int NS, bool MAP, bool PARTS>
__global__ __launch_bounds__(512, 2) void k_attn_whole(const bf16x8* __restrict__ Qp, const bf16x8* Kc, const bf16x8* Vc, bf16x8* Kt,
                                                       bf16x8* Vt, const int32_t* __restrict__ kv_len,
                                                       const uint32_t* __restrict__ anc, bf16x8* __restrict__ xp, int nh, int Tp,
                                                       int cap_blocks, float scale_log2, int stride, int nseq, int MB, PartView pv,
                                                       RowTable rt, RowRef rr, int P, float* __restrict__ opart,
                                                       float2* __restrict__ mlpart) {
    static_assert(!PARTS || FR, "parts: the last one builds the tree's keys");
    constexpr int KK = HD / 16, EB = HD / 32, NV = 2 * EB, BLK = HD * 4, NW = 8;
    constexpr int QU = KK * 2 * 64;    // 16-byte units of the queries
    constexpr int OU = EB * 4 * 64;    // of a wave's O in the merge area
    static_assert(NW * 2 * 64 * 4 <= QU * 16, "merge scalars fit the query area");
    __shared__ __attribute__((aligned(1024))) bf16x8 lds[QU + NW * OU];
    bf16x8* const qs = lds;
    bf16x8* const tkv = lds + QU;      // FR: the tree's key blocks, then its value blocks; the merge area later
    const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63, g = lane >> 5, tl = lane & 31;
    // The query blocks of a (sequence, head) lie `stride` workgroups apart, a multiple of eight: on one XCD, whose L2 then serves
    // the blocks that they all read.
    const int group = blockIdx.x / stride, combo = blockIdx.x - group * stride;
    const int part = PARTS ? group % P : 0, tg = PARTS ? group / P : group;
    if (combo >= nh * nseq) return;
    const int h = combo % nh, b = combo / nh, TB = Tp / 32;
    if (MAP && tg * 32 >= rr.map->len[b]) return;
    const int row0 = MAP ? rr.map->off[b] : b * rr.R, row_last = (MAP ? rr.map->len[b] : rr.R) - 1;
    const int sq = MAP ? rr.map->seq[b] : b;
    // blocks of the tree up to the rows' own (later ones hold no ancestors); the last part has them
    const int ntree = !PARTS || part == P - 1 ? tg + 1 : 0;
    uint4 ancq[AW / 4];
#pragma unroll
    for (int q = 0; q < AW / 4; ++q) ancq[q] = *(const uint4*)(anc + ((size_t)b * Tp + tg * 32 + tl) * SD_ANC_WORDS + 4 * q);
    const int n = MAP ? rr.map->ctx[b] : kv_len[sq];
    const bf16x8* kcb = Kc + ((size_t)sq * nh + h) * cap_blocks * BLK + lane;
    const bf16x8* vcb = Vc + ((size_t)sq * nh + h) * cap_blocks * BLK + lane;
    const size_t thead = ((size_t)b * nh + h) * TB * BLK;

    // Items: the cache's blocks, then the tree's. The waves take equal runs of them. With FR the tree's are in LDS: a wave that
    // has some comes to them after its cache blocks, when its registers are free.
    // PARTS: this part's share [b0, nblk) of the sequence's blocks, the tree's counted in.
    int nblk = (n + 31) >> 5, b0 = 0;
    if constexpr (PARTS) {
        const int each = (nblk + tg + 1 + P - 1) / P;
        b0 = min(part * each, nblk);
        nblk = part == P - 1 ? nblk : min(b0 + each, nblk);
    }
    const int total = nblk - b0 + ntree, base = total / NW, more = total - base * NW;
    const int j0 = __builtin_amdgcn_readfirstlane(b0 + wave * base + min(wave, more));
    const int j1 = j0 + base + (wave < more ? 1 : 0);
    const int je = FR ? max(j0, min(j1, nblk)) : j1;   // items [j0, je) come from memory
    auto kaddr = [&](int j) -> const bf16x8* {
        return FR || j < nblk ? kcb + (size_t)min(j, cap_blocks - 1) * BLK : Kt + thead + (size_t)(j - nblk) * BLK + lane;
    };
    auto vaddr = [&](int j) -> const bf16x8* {
        return FR || j < nblk ? vcb + (size_t)min(j, cap_blocks - 1) * BLK : Vt + thead + (size_t)(j - nblk) * BLK + lane;
    };
    bf16x8 kr[KK], vr[NV];
    auto request_k = [&](int j) {
        const bf16x8* p = kaddr(j);
#pragma unroll
        for (int i = 0; i < KK; ++i) kr[i] = __builtin_nontemporal_load(p + i * 64);
    };
    auto request_v = [&](int j) {
        const bf16x8* p = vaddr(j);
#pragma unroll
        for (int i = 0; i < NV; ++i) vr[i] = __builtin_nontemporal_load(p + i * 64);
    };
    const int jf = min(j0, max(je - 1, 0));            // (a wave without such items: a block in bounds, unused)
    request_k(jf);
    request_v(jf);

    if constexpr (FR) {
        constexpr int NA = HD / 16;                    // pieces of 8 dims + their rotary partners per row
        auto row_of = [&](int t) { return row0 + min(t, row_last); };
        float r1[8], r2[8];
        for (int it = tid; it < ntree * 2 * 32 * NA; it += NW * 64) {
            const int blk = it / (2 * 32 * NA), rem = it - blk * (2 * 32 * NA), which = 1 + rem / (32 * NA), a = rem % NA;
            const int t = blk * 32 + (rem % (32 * NA)) / NA;
            rope_kv_values<true, NS>(pv, rt, nh, HD, which, h, a, row_of(t), r1, r2);
            if (which == 1) {
                bf16x8 k1, k2;
#pragma unroll
                for (int i = 0; i < 8; ++i) { k1[i] = (__bf16)r1[i]; k2[i] = (__bf16)r2[i]; }
                const int u1 = (int)(kblk_index(t, a * 8, HD) >> 3), u2 = (int)(kblk_index(t, HD / 2 + a * 8, HD) >> 3);
                tkv[u1] = k1;
                tkv[u2] = k2;
                if (blk == tg) { Kt[thead + u1] = k1; Kt[thead + u2] = k2; }
            } else {
                __bf16 *lv = (__bf16*)(tkv + ntree * BLK), *gv = (__bf16*)(Vt + thead);
#pragma unroll
                for (int i = 0; i < 8; ++i) {
                    const int e1 = (int)vblk_index(t, a * 8 + i, HD), e2 = (int)vblk_index(t, HD / 2 + a * 8 + i, HD);
                    lv[e1] = (__bf16)r1[i];
                    lv[e2] = (__bf16)r2[i];
                    if (blk == tg) { gv[e1] = (__bf16)r1[i]; gv[e2] = (__bf16)r2[i]; }
                }
            }
        }
        if (tid < 32 * NA) {                           // (half of the threads at head_dim 128)
            const int t = tid / NA, a = tid % NA;
            rope_kv_values<true, NS>(pv, rt, nh, HD, 0, h, a, row_of(tg * 32 + t), r1, r2);
            bf16x8 hi, lo;
            split_hilo(r1, hi, lo);
            const int u1 = (int)(qblk_index(t, a * 8, HD) >> 3), u2 = (int)(qblk_index(t, HD / 2 + a * 8, HD) >> 3);
            qs[u1] = hi;
            qs[u1 + 64] = lo;
            split_hilo(r2, hi, lo);
            qs[u2] = hi;
            qs[u2 + 64] = lo;
        }
    } else {
        const bf16x8* qsrc = Qp + (((size_t)b * nh + h) * TB + tg) * QU;
#pragma unroll
        for (int i = 0; i < (QU + NW * 64 - 1) / (NW * 64); ++i) {
            const int u = i * NW * 64 + tid;
            if (QU % (NW * 64) == 0 || u < QU) qs[u] = qsrc[u];
        }
    }

    f32x16 O[EB], S;
    float mrun = NEG_INF, lrun = 0.f;
#pragma unroll
    for (int eb = 0; eb < EB; ++eb)
#pragma unroll
        for (int v = 0; v < 16; ++v) O[eb][v] = 0.f;
    __syncthreads();                                   // queries (and the tree's blocks) are in LDS

    auto qk = [&]() {
        int ql = lane;
        asm volatile("" : "+v"(ql));                   // keep the query reads in the loop
        bf16x8 st[3][2];
        auto stage = [&](int si, int kk) {
            st[si][0] = qs[(kk * 2) * 64 + ql];
            st[si][1] = qs[(kk * 2 + 1) * 64 + ql];
        };
        stage(0, 0);
        stage(1, 1);
#pragma unroll
        for (int v = 0; v < 16; ++v) S[v] = 0.f;
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
            if (kk + 2 < KK) stage((kk + 2) % 3, kk + 2);
            __builtin_amdgcn_sched_barrier(0);
            S = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kr[kk], st[kk % 3][0], S, 0, 0, 0);
            S = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kr[kk], st[kk % 3][1], S, 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    auto softmax_pv = [&](int j) {
        const bool tr = j >= nblk;
        const int blk = tr ? j - nblk : j, left = n - blk * 32;
        bf16x8 pf[2], pl[2];
        if (tr || left < 32) {                         // (wave-uniform)
            uint32_t vis;
            if (tr) {
                uint4 aq = ancq[0];
                if constexpr (AW == 8) {
                    const bool up = (blk & 4) != 0;
                    aq.x = up ? ancq[1].x : aq.x; aq.y = up ? ancq[1].y : aq.y;
                    aq.z = up ? ancq[1].z : aq.z; aq.w = up ? ancq[1].w : aq.w;
                }
                const uint64_t lo64 = aq.x | ((uint64_t)aq.y << 32), hi64 = aq.z | ((uint64_t)aq.w << 32);
                vis = (uint32_t)(((blk & 2) ? hi64 : lo64) >> ((blk & 1) * 32));       // word blk of the row's ancestor set
            } else vis = (1u << left) - 1u;
            vis >>= 4 * g;                             // lane (t = tl, g) holds rows 8 (v / 4) + 4 g + v % 4 of the block
#pragma unroll
            for (int v = 0; v < 16; ++v) S[v] = (vis & (1u << (8 * (v >> 2) + (v & 3)))) ? S[v] : NEG_INF;
        }
        float mx = S[0];
#pragma unroll
        for (int v = 1; v < 16; ++v) mx = fmaxf(mx, S[v]);
        mx = fmaxf(mx, __shfl_xor(mx, 32)) * scale_log2;
        const bool upd = mx > mrun + LAZY_MAX;
        if (__any(upd)) {
            const float alpha = upd ? __builtin_amdgcn_exp2f(mrun - mx) : 1.f;
            mrun = upd ? mx : mrun;
            lrun *= alpha;
#pragma unroll
            for (int eb = 0; eb < EB; ++eb)
#pragma unroll
                for (int v = 0; v < 16; ++v) O[eb][v] *= alpha;
        }
        const float muse = (mrun == NEG_INF) ? 0.f : mrun;
        float psum = 0.f;
#pragma unroll
        for (int p = 0; p < 2; ++p)
#pragma unroll
            for (int s = 0; s < 8; ++s) {
                const float e = __builtin_amdgcn_exp2f(__builtin_fmaf(S[8 * p + s], scale_log2, -muse));
                psum += e;
                const __bf16 hi = (__bf16)e;
                pf[p][s] = hi;
                pl[p][s] = (__bf16)(e - (float)hi);
            }
        lrun += psum;
#pragma unroll
        for (int p = 0; p < 2; ++p) {
#pragma unroll
            for (int eb = 0; eb < EB; ++eb) O[eb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vr[p * EB + eb], pf[p], O[eb], 0, 0, 0);
#pragma unroll
            for (int eb = 0; eb < EB; ++eb) O[eb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vr[p * EB + eb], pl[p], O[eb], 0, 0, 0);
        }
    };
    for (int j = j0; j < je; ++j) {
        const int nx = min(j + 1, je - 1);             // past the wave's last: that one again
        qk();
        request_k(nx);
        softmax_pv(j);
        request_v(nx);
    }
    if constexpr (FR) {
        for (int j = max(j0, nblk); j < j1; ++j) {
            const bf16x8 *kp = tkv + (j - nblk) * BLK + lane, *vp = tkv + (ntree + j - nblk) * BLK + lane;
#pragma unroll
            for (int i = 0; i < KK; ++i) kr[i] = kp[i * 64];
#pragma unroll
            for (int i = 0; i < NV; ++i) vr[i] = vp[i * 64];
            qk();
            softmax_pv(j);
        }
    }

    // The waves' contributions meet: O tiles in the merge area, (max, sum) in the query area; each wave finishes EB * 4 / NW of
    // the 4 x 64-lane pieces of the result.
    float4* mo = (float4*)(lds + QU);                  // [wave][piece = eb * 4 + i][lane]
    float* mml = (float*)lds;                          // [wave][2][64]
    __syncthreads();                                   // everybody is done with the queries and the tree's blocks
#pragma unroll
    for (int eb = 0; eb < EB; ++eb)
#pragma unroll
        for (int i = 0; i < 4; ++i)
            mo[wave * OU + (eb * 4 + i) * 64 + lane] = make_float4(O[eb][4 * i], O[eb][4 * i + 1], O[eb][4 * i + 2], O[eb][4 * i + 3]);
    mml[(wave * 2 + 0) * 64 + lane] = mrun;
    mml[(wave * 2 + 1) * 64 + lane] = lrun;
    __syncthreads();
    float sc[NW], M = NEG_INF, L = 0.f;
#pragma unroll
    for (int w = 0; w < NW; ++w) { sc[w] = mml[(w * 2) * 64 + lane]; M = fmaxf(M, sc[w]); }
    const float Muse = (M == NEG_INF) ? 0.f : M;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        sc[w] = exp2f(sc[w] - Muse);                   // exp2(-inf) = 0 for a wave that saw nothing
        L += sc[w] * mml[(w * 2 + 1) * 64 + lane];
    }
    L += __shfl_xor(L, 32);
    const float inv = L > 0.f ? 1.f / L : 0.f;
    const int t = tg * 32 + tl;
    const size_t prow = (((size_t)b * nh + h) * P + part) * Tp + t;      // (PARTS)
    if (PARTS && wave == 0 && g == 0 && t <= row_last) mlpart[prow] = make_float2(M, L);
#pragma unroll
    for (int q = 0; q < EB * 4 / NW; ++q) {
        const int piece = wave * (EB * 4 / NW) + q;    // dims 8 piece + 4 g ..
        float f[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const float4 x = mo[w * OU + piece * 64 + lane];
            f[0] += sc[w] * x.x; f[1] += sc[w] * x.y; f[2] += sc[w] * x.z; f[3] += sc[w] * x.w;
        }
        if (t > row_last) continue;
        if constexpr (PARTS) {
            *(float4*)(opart + prow * HD + piece * 8 + 4 * g) = make_float4(f[0], f[1], f[2], f[3]);
            continue;
        }
        bf16x4 hi, lo;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float v = f[i] * inv;
            hi[i] = (__bf16)v;
            lo[i] = (__bf16)(v - (float)hi[i]);
        }
        const int m = row0 + t, k = h * HD + piece * 8;
        uint16_t* out = (uint16_t*)xp + xpack_index(m, k, MB) + 4 * g;
        *(bf16x4*)out = hi;
        *(bf16x4*)(out + XPART) = lo;
    }
}

void launch_attn_whole(const void* q_packed, const void* kc, const void* vc, void* kt, void* vt, const int32_t* kv_len,
                       const uint32_t* anc, void* x_packed, RowRef rr, int B, int nh, int hd, int Tp, int cap_blocks, int MB,
                       hipStream_t s, hipEvent_t ev0, hipEvent_t ev1, const PartView* qkv, const RowTable* rt, int P, float* opart,
                       float2* mlpart) {
    const float scale_log2 = 1.4426950408889634f / sqrtf((float)hd);
    const int stride = (nh * B + 7) / 8 * 8, TG = Tp / 32;
    const PartView pv = qkv ? *qkv : PartView{nullptr, 0, 0, nullptr, 0};
    const RowTable rta = rt ? *rt : RowTable{nullptr, nullptr, nullptr, nullptr};
#define AW_ARGS (const bf16x8*)q_packed, (const bf16x8*)kc, (const bf16x8*)vc, (bf16x8*)kt, (bf16x8*)vt, kv_len, anc, (bf16x8*)x_packed, \
                nh, Tp, cap_blocks, scale_log2, stride, B, MB, pv, rta, rr, P, opart, mlpart
#define AW_GOP(HD_, AW_, FR_, NS_, MAP_, PARTS_)                                                                                 \
    do {                                                                                                                         \
        const dim3 grid(stride * TG * (PARTS_ ? P : 1));                                                                         \
        if (ev0 || ev1)                                                                                                          \
            hipExtLaunchKernelGGL((k_attn_whole<HD_, AW_, FR_, NS_, MAP_, PARTS_>), grid, dim3(512), 0, s, ev0, ev1, 0, AW_ARGS); \
        else                                                                                                                     \
            hipLaunchKernelGGL((k_attn_whole<HD_, AW_, FR_, NS_, MAP_, PARTS_>), grid, dim3(512), 0, s, AW_ARGS);                 \
    } while (0)
    // (parts: two row blocks per sequence, whose queries and tree keys this launch always makes itself: FR)
#define AW_GO(HD_, AW_, FR_, NS_, MAP_)                                                                                          \
    do {                                                                                                                         \
        if (FR_ && P > 1) AW_GOP(HD_, AW_, FR_, NS_, MAP_, FR_ != 0);                                                            \
        else AW_GOP(HD_, AW_, FR_, NS_, MAP_, false);                                                                            \
    } while (0)
#define AW_MAP(HD_, AW_, FR_, NS_) do { if (rr.map) AW_GO(HD_, AW_, FR_, NS_, true); else AW_GO(HD_, AW_, FR_, NS_, false); } while (0)
#define AW_HD(HD_)                                                                                                               \
    do {                                                                                                                         \
        if (qkv && !qkv->cnt && qkv->nmax == 4) AW_MAP(HD_, 4, 1, 4);                                                            \
        else if (qkv) AW_MAP(HD_, 4, 1, 0);                                                                                      \
        else if (Tp > 128) AW_MAP(HD_, 8, 0, 0);                                                                                 \
        else AW_MAP(HD_, 4, 0, 0);                                                                                               \
    } while (0)
    if (hd == 128) AW_HD(128); else AW_HD(64);
#undef AW_HD
#undef AW_MAP
#undef AW_GO
#undef AW_GOP
#undef AW_ARGS
}
