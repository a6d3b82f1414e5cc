// Weight-streaming GEMM for the verifying forward pass: out[m][n] = sum_k X[m][k] * W[n][k].
//
// The tree has T <= 256 rows, so every projection of the step (QKV, O, gate/up, down, LM
// head, draft heads) multiplies a few 32-row blocks of activations by a weight matrix that is
// read exactly once: the kernel is bound by the HBM read of W, not by the matrix cores. The
// design therefore (1) stores W pre-tiled as 1 KiB MFMA fragments, contraction-block-major
// ([kb][nb]): a wave fetches a fragment with one 16-byte-per-lane load, and at any moment the
// waves of the whole grid read one contiguous region of HBM, (2) keeps a ring of such loads in
// flight per wave, refilled as it is consumed, (3) shares the small activation operand between
// the waves of a workgroup through LDS, and (4) splits the contraction across workgroups so
// that every workgroup streams the same number of weight bytes (over all 256 CUs, or over fewer
// when that lets every workgroup stay inside one column group: gemm_plan_make); the consumer
// kernel sums the split partial results (deterministic, no atomics).
//
// Precision: the weights are bf16 by definition, the activations are not. Since the matrix
// cores idle most of the time in an HBM-bound kernel, each activation enters as a two-term
// bf16 expansion x = hi + lo (two MFMAs per weight fragment), which keeps ~16 mantissa bits
// of x and makes the product exact up to fp32 accumulation.
#include <type_traits>

#include "sd_internal.h"
#include "sk_gemm.h"

// ------------------------------------------------------------------------------------------
// Re-tile a row-major bf16 matrix W[N][K] into fragment order (see sd_internal.h).
__global__ void k_pack_weight(const uint4* __restrict__ src, uint4* __restrict__ dst, int N, int K,
                              int nb_offset, int KB, int NBsrc, int NBdst) {
    size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;   // one 16-byte piece each
    size_t total = (size_t)NBsrc * KB * 64;
    if (idx >= total) return;
    int lane = (int)(idx & 63);
    size_t t = idx >> 6;
    int kb = (int)(t % KB);
    int nb = (int)(t / KB);
    int n = nb * 32 + (lane & 31);
    int k0 = kb * 16 + (lane >> 5) * 8;
    uint4 v = make_uint4(0, 0, 0, 0);
    if (n < N) v = src[((size_t)n * K + k0) >> 3];
    dst[((size_t)kb * NBdst + nb + nb_offset) * 64 + lane] = v;
}

void launch_pack_weight(const void* src, void* dst, int N, int K, int nb_offset, int NBdst, int KB, hipStream_t s) {
    int NBsrc = (N + 31) / 32;
    size_t total = (size_t)NBsrc * KB * 64;
    int threads = 256;
    unsigned blocks = (unsigned)((total + threads - 1) / threads);
    hipLaunchKernelGGL(k_pack_weight, dim3(blocks), dim3(threads), 0, s, (const uint4*)src, (uint4*)dst, N, K,
                       nb_offset, KB, NBsrc, NBdst);
}

// ------------------------------------------------------------------------------------------
// Balanced streaming ("stream-K") over MT = 1 or 2 row blocks of 32 rows (this kernel; also the GEMM body of the
// persistent layer kernel, there with eight row blocks as well) or more (the kernel after it).
//
// The work of one GEMM is the list of units (column group of 256 outputs, contraction block),
// contraction block fastest; workgroup g of G takes the contiguous range [g*U/G, (g+1)*U/G),
// so every workgroup streams the same number of weight bytes whatever N and K are (one
// workgroup per CU: no tail round). A range touches at most a few column groups
// ("segments"); each segment's partial tile goes to slot = ordinal of the workgroup among
// the contributors of that column group, and the consumer sums cnt[group] slots in slot
// order (deterministic, no atomics).
//
// Eight waves, wave w owns columns [32*(8*group + w), +32). Every wave keeps a ring of R
// weight fragments in flight and refills a slot the moment it is consumed, across segment
// boundaries, so the HBM stream of a wave never drains before its last fragment. Segments
// are padded to a multiple of R steps with zero fragments (no loads, idle MFMA work only),
// which keeps every ring slot a compile-time register.
//
// The shared activation operand is double-buffered in LDS in chunks of XK contraction blocks.
// Loads of one wave return in order, so an activation load queues behind the HBM loads issued
// before it: chunks are therefore fetched one ring-length (R steps) ahead, by all threads, and
// parked in registers until the chunk before them has been consumed.
// (At most 128 registers, 94 in use: the next workgroup can start on a compute unit while this one ends.)
template <int MT>
__global__ __launch_bounds__(512, 4) void k_gemm_sk(const bf16x8* __restrict__ Xp, const bf16x8* __restrict__ Wp,
                                                    const bf16x8* __restrict__ zfrag, float* __restrict__ out,
                                                    int KB, int NB, int ldo, size_t slot_stride, int rows, int upw, int rem,
                                                    uint32_t kb_magic, const int32_t* __restrict__ slot0_tab, OperandTouch touch) {
    __shared__ bf16x8 xs[SK_LDS_UNITS];
    SkGemm<MT> gm;
    gm.setup(Xp, Wp, zfrag, out, KB, NB, ldo, slot_stride, rows, upw, rem, kb_magic, slot0_tab, blockIdx.x, gridDim.x);
    uint32_t t = 0;
    if (touch.shares) t = touch_operand(Xp + (size_t)gm.cur.kb * SkGemm<MT>::PER_KB, upw * SkGemm<MT>::PER_KB * 16, touch);
    gm.issue_x();                                      // the short L2 loads first: a wave's loads return in order
    gm.issue_ring();
    gm.template run<false>(xs, SkRowScale{nullptr, 0, 0.f, 0.f}, nullptr);
    touched(t);
}

// ------------------------------------------------------------------------------------------
// Four row blocks and more, with the operand roles swapped: the WEIGHT fragments of a step go through LDS and the activations
// stay in registers. With many row blocks the kernel above reads every activation fragment from LDS once per column block, and
// the LDS port and the matrix cores are both needed all the time. Here a tile is MT row blocks x CG column blocks for four waves;
// a wave has two row blocks and all of the columns (MT = 8) or half of them (MT = 4): its activations come straight from L2 into
// registers, and every weight fragment that it reads from LDS feeds four products.
//
// Workgroup g = column group g / S, segment g % S of the contraction: one partial tile each, slot = segment. The width of a
// group is chosen with the split (gemm_plan_rows, gemm_plan_prompt). In a prompt pass there are RT tiles of rows: workgroups
// go to the XCDs round-robin, so the RT tiles of a (column group, segment) are dealt to one XCD, next to one another, and the
// weights come from memory once. A last tile may reach past the operand's MB row blocks; those products are not stored.
//
// A wave alone on its SIMD issues everything itself, so loads, LDS reads and writes go one by one between the products, evenly
// (a wave cannot issue past a load that the address unit has not taken yet). Per iteration (two contraction blocks), a quarter
// being the products of one block and one term: the next iteration's weight fragments go to the other LDS buffer, the second
// block's are read; barrier; the next first block's are read; every quarter asks for what the quarter before it has done with.
// 1890 cycles per iteration of eight row and six column blocks, 1536 of them products; 1490 of 1024 at four by eight.
// What bounds it is the card's power: at that pace the clock is 1.63 GHz on dense data and 2.29 on zeros (QKV of 1024 rows, the
// loop alone, 148 and 106 us), products alone run at 1.83. Bytes moved are therefore time even where no unit is full: without
// the activations' loads 127 us, without the weights' 129, without LDS 119, without any of them 106.
// It replaced one of eight waves with a row block each (two products per fragment, a barrier per contraction block): 7B shape,
// eight 32-node trees 1481 -> 1411 us, ten heads and 256 nodes 1275 -> 1212; 13B shape, 128 nodes 1255 -> 1209; a 256-row launch of
// gate/up 84.0 -> 81.4, of down 43.8 -> 42.3, a 128-row launch of the 13B shape's gate/up 76.1 -> 72.1. Prompts, four layers, 1500
// tokens: 5483 -> 5017, of which a part is the next two paragraphs' (gate/up and SwiGLU of 1024 rows 346 -> 289, down 200 -> 180).
// Not kept: gate/up of 256 rows with whole sums, in tiles of eight by four (88 us; 77 and 11 for SwiGLU).
//
// chain (TILE_PROMPT, TILE_SWIGLU): every so many contraction blocks (a multiple of eight, the loop's grain is four) the products
// are added to a second set and begin again at zero: see gemm_plan_prompt. Eight of its blocks are in LDS; the other four of the
// tile of six columns are in registers (3 us a fold at 1024 rows), the other eight of the tile of eight in the output, where the
// sums end up anyway (registers for half of those spill: down projection 233 us for 180).
//
// TILE_SWIGLU (gate/up with whole sums, gemm_plan_swiglu): half of a group's columns are gate columns, half the up columns that
// belong to them; the workgroup writes silu(gate) * up as the next projection's operand. The sums, 90 MB at 1024 rows of the 7B
// shape, are neither written nor read, and a launch of 23 us is gone.
enum { TILE_STEP, TILE_PROMPT, TILE_SWIGLU };
template <int MT, int CG, int KIND>
__global__ __launch_bounds__(256, 1) void k_gemm_tile(const bf16x8* __restrict__ Xp, const bf16x8* __restrict__ Wp,
                                                      void* __restrict__ out_, int KB, int NB, int ldo, size_t slot_stride, int rows,
                                                      int S, int MB, int RT, int n_combo, int chain, int KBf) {
    constexpr bool SWIGLU = KIND == TILE_SWIGLU, CHAINS = KIND != TILE_STEP;
    constexpr int DW = 2;                              // iterations whose weights are in flight (four: steps 0.6-1.2 % slower)
    static_assert(MT == 8 || (MT == 4 && !SWIGLU), "four waves of two row blocks each, or two beside two");
    constexpr int RW = MT / 2, CPW = CG * MT / 8;      // waves one above the other; column blocks of a wave
    constexpr int NF = 2 * CPW, LW = CG / 2;           // product blocks of a wave; weight fragments that it loads per iteration
    // the second set of sums: blocks in LDS, in registers, in the output (beyond what there is room for)
    constexpr int NL = !CHAINS ? 0 : NF < 8 ? NF : 8, NN = CHAINS && NF == 12 ? 4 : 0, NM = CHAINS ? NF - NL - NN : 0;
    static_assert(NM >= 0 && !(SWIGLU && NM), "an operand has no room for sums");
    __shared__ bf16x8 ws[2][2 * CG * 64];
    __shared__ f32x4 far[NL ? NL * 4 : 1][NL ? 256 : 1];               // (every thread its own)
    // (wave in a scalar register: what follows from it is the same in all lanes)
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const int q = blockIdx.x >> 3, tile = q % RT, combo = (q / RT) * 8 + (blockIdx.x & 7);
    if (combo >= n_combo) return;
    const int rb = tile * MT + wave % RW * 2;          // this wave's row blocks: rb and rb + 1
    const int c0 = wave / RW * CPW;                    // ... and its first column block of the group's
    const int ng = combo / S, seg = combo - ng * S;
    const int n = KB / S, kb0 = seg * n, NI = (n + 1) / 2, len = CHAINS && chain ? chain / 2 : NI + DW;
    // column block j of the group: neighbours, or (SWIGLU) half of them gate blocks and half the up blocks that belong to them
    const int half = NB >> 1;
    auto column = [&](int j) {
        if constexpr (!SWIGLU) return ng * CG + j;
        else return j < CG / 2 ? ng * (CG / 2) + j : half + ng * (CG / 2) + j - CG / 2;
    };
    const uint32_t xstep = (uint32_t)MB * 2048u;       // bytes of a contraction block
    const uint32_t wstep = (uint32_t)NB * 1024u;
    uint32_t wv[LW], xv[2];                            // this lane's bytes in an iteration's weights and activations
#pragma unroll
    for (int l = 0; l < LW; ++l) {                     // fragment f: contraction block f / CG, column block f % CG
        const int f = wave + 4 * l;
        wv[l] = (uint32_t)(f / CG) * wstep + (uint32_t)min(column(f % CG), NB - 1) * 1024u + lane * 16;
    }
#pragma unroll
    for (int k = 0; k < 2; ++k) xv[k] = (uint32_t)k * xstep + (uint32_t)rb * 2048u + lane * 16;
    const char *wb = (const char*)(Wp + (size_t)kb0 * NB * 64), *xb = (const char*)(Xp + (size_t)kb0 * MB * 128);
    // an iteration's bytes up to the end of the segment: what lies past it is read as zeros
    // (32-bit scalar arithmetic, and words that are scalars to the compiler: it would step through the lanes' resources)
    const int wmost = 0x7fffffff / (int)wstep, xmost = 0x7fffffff / (int)xstep;
    auto bytes = [&](const char* base, int it, uint32_t step, int most) {
        return __builtin_amdgcn_make_buffer_rsrc((void*)TileStore::uniform(base + (size_t)it * 2 * step), 0,
                                                 __builtin_amdgcn_readfirstlane(max(min(n - 2 * it, most), 0) * (int)step), 0x00020000);
    };
    auto wfrag = [&](__amdgpu_buffer_rsrc_t r, int l) {
        return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(r, wv[l], 0, /*nontemporal*/ 2));
    };
    auto xfrag = [&](__amdgpu_buffer_rsrc_t r, int k, int t, int p) {
        return __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(r, xv[k] + t * 2048 + p * 1024, 0, 0));
    };
    f32x16 near[NN ? NN : 1], acc[2][CPW];
#pragma unroll
    for (int f = 0; f < NN; ++f) near[f] = f32x16{0.f};
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int j = 0; j < CPW; ++j) acc[t][j] = f32x16{0.f};
    bf16x8 w[DW][LW], x[2][2][2][2], b[2][CPW];         // x: [iteration][contraction block][row block][hi, lo]
#pragma unroll
    for (int i = 0; i < DW; ++i) {
        const auto wr = bytes(wb, i, wstep, wmost), xr = bytes(xb, i, xstep, xmost);
#pragma unroll
        for (int l = 0; l < LW; ++l) w[i][l] = wfrag(wr, l);
        if (i < 2)
#pragma unroll
        for (int k = 0; k < 2; ++k)
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int p = 0; p < 2; ++p)
                    if (i == 0 || k == 0 || p == 0) x[i & 1][k][t][p] = xfrag(xr, k, t, p);
    }
    if (CHAINS && chain)                               // (workgroup-uniform)
#pragma unroll
        for (int i = 0; i < NL * 4; ++i) far[i][tid] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int l = 0; l < LW; ++l) ws[0][(wave + 4 * l) * 64 + lane] = w[0][l];
    __syncthreads();
#pragma unroll
    for (int j = 0; j < CPW; ++j) b[0][j] = ws[0][(c0 + j) * 64 + lane];
    {
        const auto wr = bytes(wb, DW, wstep, wmost);
#pragma unroll
        for (int l = 0; l < LW; ++l) w[0][l] = wfrag(wr, l);
    }
    // block f of the wave's sums in the output
    const int gq = lane >> 5;
    auto store_at = [&](int f) {
        return TileStore((float*)out_ + (size_t)seg * slot_stride, (rb + f / CPW) * 32, rows, ldo);
    };
    auto offset = [&](int f, int v, int g, int ld) {
        return ((8 * (v >> 2) + 4 * g + (v & 3)) * ld + column(c0 + f % CPW) * 32 + (lane & 31)) * 4;
    };
    constexpr int AHEAD = 6;                           // pieces of four sums read before they are added to
    f32x4 o[AHEAD];
    auto fetch = [&](int i) {
        if (i < NL * 4) o[i % AHEAD] = far[i < NL * 4 ? i : 0][tid];
    };
    auto xr_old = bytes(xb, 1, xstep, xmost);                 // (the last quarter of an iteration's activations is asked for in the next one)
    for (int i0 = 0;;) {                               // a chain: iterations [i0, i1)
        const int i1 = min(i0 + len, NI);
        for (; i0 < i1; i0 += DW) {
#pragma unroll
            for (int iu = 0; iu < DW; ++iu) {
                const int it = i0 + iu, ii = iu & 1, buf = ii ^ 1, nx = ii ^ 1, nw = (iu + 1) % DW;      // (LDS buffers, ring slots)
                const auto wr = bytes(wb, it + 1 + DW, wstep, wmost), xr = bytes(xb, it + 2, xstep, xmost);
                // the products of one contraction block and one term, n_ops other things spread evenly among them
                auto quarter = [&](int k, int p, int n_ops, auto&& op) {
#pragma unroll
                    for (int i = 0; i < NF; ++i) {
                        acc[i & 1][i >> 1] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[ii][k][i & 1][p], b[k][i >> 1], acc[i & 1][i >> 1], 0, 0, 0);
#pragma unroll
                        for (int u = 0; u < n_ops; ++u)
                            if ((2 * u + 1) * NF / (2 * n_ops) == i) {
                                __builtin_amdgcn_sched_barrier(0);
                                op(u);
                                __builtin_amdgcn_sched_barrier(0);
                            }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                };
                constexpr int W1 = LW / 3, W2 = (LW - W1) / 2, W3 = LW - W1 - W2;     // weight loads of the last three quarters
                constexpr int B1 = CPW / 2, B2 = CPW - B1;
                quarter(0, 0, LW + 2 + CPW, [&](int u) {
                    if (u < LW) ws[buf][(wave + 4 * u) * 64 + lane] = w[nw][u];       // (its readers passed the previous barrier)
                    else if (u < LW + 2) x[nx][1][u - LW][1] = xfrag(xr_old, 1, u - LW, 1);
                    else b[1][u - LW - 2] = ws[ii][(CG + c0 + u - LW - 2) * 64 + lane];
                });
                quarter(0, 1, 2 + W1, [&](int u) {
                    if (u < 2) x[ii][0][u][0] = xfrag(xr, 0, u, 0);
                    else w[nw][u - 2] = wfrag(wr, u - 2);
                });
                __syncthreads();
                __builtin_amdgcn_sched_barrier(0);
                quarter(1, 0, 2 + W2 + B1, [&](int u) {
                    if (u < 2) x[ii][0][u][1] = xfrag(xr, 0, u, 1);
                    else if (u < 2 + W2) w[nw][W1 + u - 2] = wfrag(wr, W1 + u - 2);
                    else b[0][u - 2 - W2] = ws[buf][(c0 + u - 2 - W2) * 64 + lane];
                });
                quarter(1, 1, 2 + W3 + B2, [&](int u) {
                    if (u < 2) x[ii][1][u][0] = xfrag(xr, 1, u, 0);
                    else if (u < 2 + B2) b[0][B1 + u - 2] = ws[buf][(c0 + B1 + u - 2) * 64 + lane];
                    else w[nw][W1 + W2 + u - 2 - B2] = wfrag(wr, W1 + W2 + u - 2 - B2);
                });
                xr_old = xr;
            }
        }
        if (!CHAINS || i1 >= NI) break;
        const bool first = i1 == len;                  // (the first fold: nothing in the output yet)
#pragma unroll
        for (int i = 0; i < AHEAD; ++i) fetch(i);
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            f32x16 a = acc[f / CPW][f % CPW];
            asm volatile("" : "+a"(a));                // (not read before its turn)
            if (f < NL) {
#pragma unroll
                for (int z = 0; z < 4; ++z) {
                    const int i = f * 4 + z;
                    far[f < NL ? i : 0][tid] = o[i % AHEAD] + f32x4{a[4 * z], a[4 * z + 1], a[4 * z + 2], a[4 * z + 3]};
                    fetch(i + AHEAD);
                    __builtin_amdgcn_sched_barrier(0);
                }
            } else if (f < NL + NN) {
                near[f < NL || f >= NL + NN ? 0 : f - NL] += a;
            } else {
                int g = gq, ld = ldo;
                asm volatile("" : "+v"(g), "+s"(ld));
                const TileStore ts = store_at(f);
                if (!first)
#pragma unroll
                    for (int v = 0; v < 16; ++v) a[v] += ts.get(offset(f, v, g, ld));
                if (column(c0 + f % CPW) < NB)
#pragma unroll
                    for (int v = 0; v < 16; ++v) ts.put(a[v], offset(f, v, g, ld));
            }
            acc[f / CPW][f % CPW] = f32x16{0.f};
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    auto finish = [&](auto folded_) {                  // block by block: few registers
        constexpr bool FOLDED = decltype(folded_)::value;
        if constexpr (FOLDED && !SWIGLU)
#pragma unroll
            for (int i = 0; i < AHEAD; ++i) fetch(i);
        auto total = [&](int f) {                      // block f of the sums, the chains folded away before included
            f32x16 a = acc[f / CPW][f % CPW];
            asm volatile("" : "+a"(a));                // (not read before its turn)
            if constexpr (FOLDED)
#pragma unroll
                for (int z = 0; z < 4; ++z) {
                    const int i = f * 4 + z;
                    if (SWIGLU && f < NL) o[i % AHEAD] = far[f < NL ? i : 0][tid];       // (not in the order of the blocks)
                    if (f < NL + NN)
#pragma unroll
                        for (int v = 0; v < 4; ++v) a[4 * z + v] += f < NL ? o[i % AHEAD][v] : near[f < NL || f >= NL + NN ? 0 : f - NL][4 * z + v];
                    if (!SWIGLU && f < NL) fetch(i + AHEAD);
                }
            return a;
        };
        if constexpr (!SWIGLU) {
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                f32x16 a = total(f);
                int g = gq, ld = ldo;                  // opaque, as in k_gemm_sk: no hoisted row offsets
                asm volatile("" : "+v"(g), "+s"(ld));
                const TileStore ts = store_at(f);
                if (f >= NL + NN && FOLDED)
#pragma unroll
                    for (int v = 0; v < 16; ++v) a[v] += ts.get(offset(f, v, g, ld));
                if (column(c0 + f % CPW) < NB)
#pragma unroll
                    for (int v = 0; v < 16; ++v) ts.put(a[v], offset(f, v, g, ld));
                __builtin_amdgcn_sched_barrier(0);
            }
        } else {
            // silu(gate) * up, block by block through LDS (a wave's own 4 KiB) into the fragments of the next projection's
            // operand: two contraction blocks x (hi, lo), written whole
            __syncthreads();                           // everybody is done with the weights
            __bf16* turn = (__bf16*)ws + wave * 2048;
            const bf16x8* turned = (const bf16x8*)turn;
#pragma unroll
            for (int t = 0; t < 2; ++t)
#pragma unroll
                for (int j = 0; j < CG / 2; ++j) {
                    const f32x16 gt = total(t * CG + j), up = total(t * CG + j + CG / 2);
                    const int c = lane & 31;           // column: contraction block c / 16 of the two, lane group c / 8 % 2, element c % 8
                    int at0 = (c >> 4) * 1024 + 32 * ((c >> 3) & 1) * 8 + (c & 7) + 4 * gq * 8;
                    asm volatile("" : "+v"(at0));
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const float y = gt[v] / (1.f + __expf(-gt[v])) * up[v];
                        const int at = at0 + (8 * (v >> 2) + (v & 3)) * 8;
                        const __bf16 hi = (__bf16)y;
                        turn[at] = hi;
                        turn[at + 512] = (__bf16)(y - (float)hi);
                    }
                    __builtin_amdgcn_wave_barrier();
                    const int kb = column(j) * 2;
                    bf16x8* dst = (bf16x8*)out_ + ((size_t)kb * MB + rb + t) * 128 + lane;
#pragma unroll
                    for (int k = 0; k < 2; ++k)
                        if (rb + t < MB && column(j) < half && kb + k < KBf) {
                            dst[(size_t)k * MB * 128] = turned[k * 128 + lane];
                            dst[(size_t)k * MB * 128 + 64] = turned[k * 128 + 64 + lane];
                        }
                    __builtin_amdgcn_wave_barrier();
                    __builtin_amdgcn_sched_barrier(0);
                }
        }
    };
    if (CHAINS && chain && chain < n) finish(std::integral_constant<bool, CHAINS>{});
    else finish(std::false_type{});
}

// ------------------------------------------------------------------------------------------
// Sums the slots of selected rows only: output row (i, b), i < H, b < B, is row i*M + sel[b] of a
// row-chunked GEMM sequence; this launch covers the chunk holding rows [row0, row0 + rows) and
// writes dst row i*B + b when that row lies in it.
__global__ void k_reduce_selected(PartView pv, float* __restrict__ dst, const int32_t* __restrict__ sel, int B, int M,
                                  int row0, int rows) {
    const int c4 = (blockIdx.x * blockDim.x + threadIdx.x) * 4;
    const int i = blockIdx.y / B, b = blockIdx.y % B;
    const int s = sel[b];
    if (c4 >= pv.ld || s < 0 || s >= M) return;
    const int m = i * M + s - row0;
    if (m < 0 || m >= rows) return;
    const int n = part_count(pv, c4);
    float4 a = make_float4(0, 0, 0, 0);
    for (int sp = 0; sp < n; ++sp) {
        float4 v = *(const float4*)(pv.base + (size_t)sp * pv.slot_stride + (size_t)m * pv.ld + c4);
        a.x += v.x; a.y += v.y; a.z += v.z; a.w += v.w;
    }
    *(float4*)(dst + (size_t)blockIdx.y * pv.ld + c4) = a;
}
void launch_reduce_selected(PartView pv, float* dst, const int32_t* sel, int B, int H, int M, int row0, int rows,
                            hipStream_t s) {
    hipLaunchKernelGGL(k_reduce_selected, dim3((pv.ld / 4 + 255) / 256, H * B), dim3(256), 0, s, pv, dst, sel, B, M, row0,
                       rows);
}

// ------------------------------------------------------------------------------------------
#ifndef SK_SMALL_U
#define SK_SMALL_U (16 * SK_MAX_WG * 2)   // (column groups x contraction blocks) up to which half the workgroups are used
#endif

void gemm_plan_make(GemmPlan* p, int MB, int KB, int NB, int32_t* cnt_host, int32_t* slot0_host) {
    p->MB = MB; p->KB = KB; p->NB = NB;
    p->cnt_dev = nullptr;
    p->slot0_dev = nullptr;
    p->NG = (NB + 7) / 8;
    const int U = p->NG * KB;
    int G = U / 16;                                   // at least 16 steps each
    if (G > SK_MAX_WG) G = SK_MAX_WG;
    // (The figures below were taken with a weight ring 16 steps deep. With the ring of 4, looked at again: balanced over 256
    // workgroups plain decoding is 5 % slower, the O projection on 256 workgroups level.)
    // Prefer a split in which no workgroup's range crosses a column group: s workgroups per group with s a divisor
    // of KB. Every workgroup then has ONE segment, writes its partial tile once, at the end of its stream, and a
    // group has exactly s slots. With ranges that straddle groups a workgroup stores a tile in the middle of its
    // stream and the groups get one or two slots more (measured at the 7B shape, 64 rows: QKV 256 -> 192
    // workgroups, gate/up 256 -> 172, LM head 256 -> 252: step 5.23 -> 5.00 ms on one box; gate/up alone 5.08).
    // Taken when it keeps at least five eighths of the workgroups (seven eighths at eight row blocks, where the
    // matrix cores are short: there 192 of 256 workgroups made the GEMMs 5 % slower and the step no faster);
    // otherwise the balanced split stays.
    int aligned = 0;
    for (int sp = 1; p->NG * sp <= G; ++sp)
        if (KB % sp == 0) aligned = p->NG * sp;
    if (aligned * 8 >= G * (MB >= 8 ? 7 : 5)) G = aligned;
    // A small matrix (the O projection: 33 MB at the 7B shape) gains nothing from the last
    // doubling of workgroups but pays for it in partial tiles (measured 13.5 us with 128
    // workgroups / 8 slots against 14.9 us with 256 / 16, and the consumer reads half as much).
    if (G > SK_MAX_WG / 2 && U <= SK_SMALL_U) {
        const int sp = G / p->NG;                     // (aligned splits stay aligned when s is even)
        G = (G == aligned && sp % 2 == 0) ? G / 2 : SK_MAX_WG / 2;
    }
    if (G < 1) G = 1;
    p->G = G;
    // workgroup g takes upw units, the first `rem` workgroups one more (the kernels compute the same)
    p->upw = U / G;
    p->rem = U % G;
    for (int ng = 0; ng < p->NG; ++ng) cnt_host[ng] = 0;
    for (int g = 0; g < G; ++g) {
        const int u0 = g * p->upw + (g < p->rem ? g : p->rem), u1 = u0 + p->upw + (g < p->rem ? 1 : 0);
        const int ng0 = u0 / KB, ng1 = (u1 - 1) / KB;
        slot0_host[g] = cnt_host[ng0];                // contributors of its first column group before it
        for (int ng = ng0; ng <= ng1; ++ng) ++cnt_host[ng];
    }
    int slots = 1;
    for (int ng = 0; ng < p->NG; ++ng) slots = cnt_host[ng] > slots ? cnt_host[ng] : slots;
    p->slots = slots;
    p->uniform = 1;                                   // every column group has the same number of contributors?
    for (int ng = 0; ng < p->NG; ++ng) p->uniform &= (cnt_host[ng] == slots);
    p->CG = 0;
    p->S = 0;
    p->RT = p->MT = p->chain = 0;
    p->slots_max = slots;
    if (MB >= 4) gemm_plan_rows(p);
}

PartView launch_gemm(const GemmPlan& p, const void* Xp, const void* Wp, const void* zfrag, float* out, int rows, hipStream_t s,
                     hipEvent_t ev0, hipEvent_t ev1, void* swiglu, int swiglu_KB) {
    PartView pv;
    pv.base = out;
    pv.ld = p.NB * 32;
    pv.slot_stride = (size_t)p.MB * 32 * pv.ld;
    pv.cnt = p.uniform ? nullptr : p.cnt_dev;         // NULL: nmax slots everywhere, the consumer need not look it up
    pv.nmax = p.slots;
    const uint32_t kb_magic = (uint32_t)((0x100000000ull + (uint64_t)p.KB - 1) / (uint64_t)p.KB);
    // (aligned splits: one segment of one column group per workgroup)
    const OperandTouch touch = !p.CG && p.rem == 0 && p.KB % p.upw == 0 ? operand_touch(p.G, p.KB / p.upw) : OperandTouch{0, 0};
#define SK_ARGS (const bf16x8*)Xp, (const bf16x8*)Wp, (const bf16x8*)zfrag, out, p.KB, p.NB, pv.ld, pv.slot_stride, rows, p.upw, p.rem, kb_magic, p.slot0_dev, touch
#define SK_LAUNCH(KERNEL_, THREADS_, ...)                                                                  \
    do {                                                                                                   \
        if (ev0 || ev1)                                                                                    \
            hipExtLaunchKernelGGL(KERNEL_, dim3(p.G), dim3(THREADS_), 0, s, ev0, ev1, 0, SK_ARGS, ##__VA_ARGS__); \
        else                                                                                               \
            hipLaunchKernelGGL(KERNEL_, dim3(p.G), dim3(THREADS_), 0, s, SK_ARGS, ##__VA_ARGS__);          \
    } while (0)
    if (p.CG) {                                        // four row blocks and more: the aligned split of k_gemm_tile
        const int combos = (p.NB + p.CG - 1) / p.CG * p.S, G = p.RT ? (combos + 7) / 8 * 8 * p.RT : combos;
        pv.cnt = nullptr;
        pv.nmax = p.S;
#define TILE_GO(MT_, CG_, KIND_, OUT_)                                                                        \
    do {                                                                                                   \
        if (ev0 || ev1)                                                                                    \
            hipExtLaunchKernelGGL((k_gemm_tile<MT_, CG_, KIND_>), dim3(G), dim3(256), 0, s, ev0, ev1, 0, (const bf16x8*)Xp, \
                                  (const bf16x8*)Wp, (void*)OUT_, p.KB, p.NB, pv.ld, pv.slot_stride, rows, p.S, p.MB, p.RT ? p.RT : 1, combos, \
                                  p.chain, swiglu_KB);                                                     \
        else                                                                                               \
            hipLaunchKernelGGL((k_gemm_tile<MT_, CG_, KIND_>), dim3(G), dim3(256), 0, s, (const bf16x8*)Xp, (const bf16x8*)Wp, \
                               (void*)OUT_, p.KB, p.NB, pv.ld, pv.slot_stride, rows, p.S, p.MB, p.RT ? p.RT : 1, combos, p.chain, swiglu_KB); \
    } while (0)
        if (swiglu && gemm_plan_swiglu(p)) {           // (the caller has asked the same of the same plan)
            TILE_GO(8, 6, TILE_SWIGLU, swiglu);
            pv.nmax = 0;
            return pv;
        }
        const int key = (p.RT ? 100 + p.MT * 10 : p.MB * 10) + p.CG;
        if (key == 88) TILE_GO(8, 8, TILE_STEP, out);
        else if (key == 86) TILE_GO(8, 6, TILE_STEP, out);
        else if (key == 84) TILE_GO(8, 4, TILE_STEP, out);
        else if (key == 48) TILE_GO(4, 8, TILE_STEP, out);
        else if (key == 44) TILE_GO(4, 4, TILE_STEP, out);
        else if (key == 188) TILE_GO(8, 8, TILE_PROMPT, out);
        else if (key == 186) TILE_GO(8, 6, TILE_PROMPT, out);
        else if (key == 184) TILE_GO(8, 4, TILE_PROMPT, out);
        else if (key == 148) TILE_GO(4, 8, TILE_PROMPT, out);
        else if (key == 144) TILE_GO(4, 4, TILE_PROMPT, out);
        else pv.nmax = 0;                              // the planners make no other: nothing launched, nothing to read
#undef TILE_GO
        return pv;
    }
    switch (p.MB) {                                    // one or two row blocks
    case 1: SK_LAUNCH(k_gemm_sk<1>, 512); break;
    case 2: SK_LAUNCH(k_gemm_sk<2>, 512); break;
    default:                                           // plans are only ever made for 1, 2, 4 or 8 row blocks
        pv.nmax = 0;                                   // nothing launched, nothing for a consumer to read
        pv.cnt = nullptr;
        break;
    }
#undef SK_LAUNCH
#undef SK_ARGS
    return pv;
}
