// The weight-streaming GEMM of the verifying pass as a device function, shared by the stand-alone kernel
// (gemm.hip) and the persistent layer kernel (fused.hip). See gemm.hip for the design.
#pragma once
#include "sd_internal.h"

// Stores of one row block (rows row0 .. row0 + 31) of a partial tile of `rows` rows of ldo floats (all wave-uniform).
// Write-through: the tiles are consumed by other XCDs anyway, and lines left dirty in this XCD's L2 would only be written
// back at the end of the kernel, lengthening it. The rows of the last row block that do not exist (plain decoding: 31 of
// 32) lie past the buffer resource's size and the hardware drops their stores: no branch and no mask in the epilogue
// (written with either, the 64-row launches took 0.5 us longer each although all of their rows exist). One resource per
// row block: 32 * ldo * 4 bytes at most, a 32-bit size for every projection that fits the card. Its words are put into scalar
// registers by hand: the compiler cannot tell that they are the same in all lanes and stepped through the lanes' resources in a
// loop of twenty instructions around EVERY store (32 to 192 of them at the end of a launch). 7B shape, 64-node step of 32 layers
// 4493 -> 4472 us, prompt of 1500 tokens 5546 -> 5512; 13B shape, 128 nodes 1263 -> 1255; nothing slower.
struct TileStore {
    __amdgpu_buffer_rsrc_t rsrc;
    __device__ __forceinline__ TileStore(float* tile, int row0, int rows, int ldo)
        : rsrc(__builtin_amdgcn_make_buffer_rsrc(uniform(tile + (size_t)row0 * ldo), 0,
                                                 __builtin_amdgcn_readfirstlane(min(max(rows - row0, 0), 32) * ldo * 4), 0x00020000)) {}
    template <class T>
    static __device__ __forceinline__ T* uniform(T* p) {
        const uint64_t a = (uint64_t)p;
        return (T*)((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)a) |
                        (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(a >> 32)) << 32);
    }
    __device__ __forceinline__ float get(int byte_offset) const {           // (what this thread has put there)
        return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsrc, byte_offset, 0, /*sc1*/ 16));
    }
    __device__ __forceinline__ void put(float v, int byte_offset) const {
        __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(v), rsrc, byte_offset, 0, /*sc1*/ 16);
    }
};

struct SkIter { int kb, ng, valid, last; };

// A workgroup's walk over its unit range [u, u1) in outer iterations of R steps, without any division
// after the first position: the next iteration starts at (ng, kb), covers min(R, rest of the segment)
// steps and is the segment's last if the segment ends within it.
struct SkWalk { int u, u1, ng, kb; };
// kb_magic = ceil(2^32 / KB): u / KB = high word of u * kb_magic for every u < 2^32 / KB (units number < 2^20)
static __device__ inline SkWalk sk_walk_init(int g, int upw, int rem, int KB, uint32_t kb_magic) {
    SkWalk w;
    w.u = g * upw + (g < rem ? g : rem);               // workgroup g takes upw units, the first `rem` one more
    w.u1 = w.u + upw + (g < rem ? 1 : 0);
    w.ng = KB == 1 ? w.u : (int)__umulhi((uint32_t)w.u, kb_magic);
    w.kb = w.u - w.ng * KB;
    return w;
}
template <int R>
static __device__ inline SkIter sk_walk_next(SkWalk& w, int KB) {
    SkIter r = {0, 0, 0, 0};
    if (w.u >= w.u1) return r;
    int send = (w.ng + 1) * KB;
    if (send > w.u1) send = w.u1;
    const int len = send - w.u;
    r.kb = w.kb;
    r.ng = w.ng;
    r.valid = len < R ? len : R;
    r.last = len <= R;
    w.u += r.valid;
    w.kb += r.valid;
    if (w.kb >= KB) { w.kb = 0; ++w.ng; }
    return r;
}

// LDS the GEMM needs: two activation chunks of up to 16 fragments, and (for a GEMM that applies the deferred RMS scale
// of its rows) the per-row factors and the scratch of their reduction
#define SK_LDS_UNITS (2 * 16 * 64)
#define SK_LDS_SCALE_FLOATS (256 + 512)

// One weight-streaming GEMM of workgroup g (512 threads), in pieces, so that a caller can request the first ring of
// weight fragments long before the activations exist (the persistent layer kernel does, across a grid barrier):
//     setup()      the workgroup's unit range and first iterations (no memory traffic but one table entry)
//     issue_ring() requests the first R weight fragments of this wave
//     issue_x()    requests the activation chunks of the first iteration (they must have been written by now)
//     run()        the main loop and the partial-tile stores; every thread of the workgroup calls it
// A workgroup (or a whole launch) without units: has_work() is false, the other calls do nothing.
template <int MT>
struct SkGemm {
    static_assert(MT == 1 || MT == 2 || MT == 8, "four row blocks: k_gemm_tile only");
    // Ring depth R, and XK contraction blocks per activation chunk (a barrier each). A shallow ring: what a wave holds in
    // flight when its stream ends is still to be multiplied then, and a workgroup's steps are padded to a multiple of R.
    // Depth 16 (chunks of 8 / MT) keeps more bytes in flight and is slower: down projection of the 7B shape (43 steps a
    // workgroup) 25.6 -> 22.2 us at 64 rows and 20.8 -> 16.4 at 1 row, O 14.7 -> 13.6, QKV 26.6 -> 25.9; in turn on one
    // box, the full step of the 64-node tree 4850 -> 4739 us, four layers over 16384 rows 992 -> 976, eight sequences of
    // plain decoding 925 -> 906. Depth 8 lies between, 6 is level with 4, 2 is 17 % slower. With eight row blocks a step
    // holds 16 MFMAs and rings of 6 and 8 measured slower too.
    static constexpr int R = 4;
    static constexpr int XK = MT == 8 ? 1 : 2;      // contraction blocks per chunk
    static constexpr int CPI = R / XK;               // chunks per outer iteration (2 or 4)
    static_assert(CPI % 2 == 0, "chunk c of every iteration is in LDS buffer c & 1");
    static constexpr int XF = XK * MT * 2;           // fragments per chunk
    static constexpr int XP = (XF * 64 + 511) / 512; // 16-byte pieces per thread per chunk (one row block: half the threads)
    static constexpr int PER_KB = MT * 2 * 64;       // 16-byte units of the row blocks per contraction block

    const bf16x8 *Xp, *Wp, *zl;
    float* out;
    int KB, NB, ldo, rows, tid, wave, lane, slot0;
    const int32_t* slot0_at;
    size_t slot_stride, wstep;
    SkWalk walk;
    SkIter cur, nxt, nx2;
    bf16x8 w[R], xr[CPI][XP];

    __device__ __forceinline__ void setup(const bf16x8* __restrict__ Xp_, const bf16x8* __restrict__ Wp_,
                                          const bf16x8* __restrict__ zfrag, float* __restrict__ out_, int KB_, int NB_,
                                          int ldo_, size_t slot_stride_, int rows_, int upw, int rem, uint32_t kb_magic,
                                          const int32_t* __restrict__ slot0_tab, int g, int G) {
        Xp = Xp_; Wp = Wp_; out = out_; KB = KB_; NB = NB_; ldo = ldo_; slot_stride = slot_stride_; rows = rows_;
        tid = threadIdx.x; wave = tid >> 6; lane = tid & 63;
        wstep = (size_t)NB * 64;
        // Every load is unconditional and its result is used as loaded: a fragment past the end of a segment is
        // fetched from a 1 KiB page of zeros (zfrag) by selecting the ADDRESS. A branch around a load, or a select
        // on its result, makes the compiler wait for the whole ring (s_waitcnt vmcnt(0)) in every iteration;
        // straight-line loads are counted exactly.
        zl = zfrag + lane;
        cur = nxt = nx2 = SkIter{0, 0, 0, 0};
        slot0 = 0;
        slot0_at = slot0_tab + (g < G ? g : 0);        // read once the ring has been issued (issue_ring)
        if (g < G) {
            walk = sk_walk_init(g, upw, rem, KB, kb_magic);
            cur = sk_walk_next<R>(walk, KB);
            nxt = sk_walk_next<R>(walk, KB);
            nx2 = sk_walk_next<R>(walk, KB);
        }
    }
    __device__ __forceinline__ bool has_work() const { return cur.valid != 0; }
    __device__ __forceinline__ const bf16x8* wptr(const SkIter& I) const {
        int nb = I.ng * 8 + wave;
        if (nb >= NB) nb = NB - 1;
        return Wp + ((size_t)I.kb * NB + nb) * 64 + lane;
    }
    __device__ __forceinline__ void xload(bf16x8 (&dst)[XP], const SkIter& I, int c) const {
        int steps = I.valid - c * XK;
        steps = steps < 0 ? 0 : (steps > XK ? XK : steps);
        const int limit = steps * PER_KB;
        const bf16x8* base = Xp + (size_t)(I.kb + c * XK) * PER_KB;
#pragma unroll
        for (int p = 0; p < XP; ++p) {
            const int i = p * 512 + tid;
            dst[p] = *((i < limit) ? base + i : zl);
        }
    }
    __device__ __forceinline__ void issue_ring() {
        if (!has_work()) return;
        const bf16x8* wc = wptr(cur);
#pragma unroll
        for (int i = 0; i < R; ++i) w[i] = __builtin_nontemporal_load((i < cur.valid) ? wc + (size_t)i * wstep : zl);
        // The slot of this workgroup's first segment (later ones: 0), wanted only when that segment ends. Read here,
        // as a vector load behind the ring, so that nothing waits for it: read in setup it was a scalar load that the
        // next wait for a kernel argument also waited for, a memory round trip before the first weight was requested.
        int zero = 0;
        asm volatile("" : "+v"(zero));              // (a vector register: the load is a vector load)
        slot0 = slot0_at[zero];
    }
    __device__ __forceinline__ void issue_x() {
        if (!has_work()) return;
#pragma unroll
        for (int c = 0; c < CPI; ++c) xload(xr[c], cur, c);
    }

    // SCALE: apply the deferred row scale sc; lds_f: SK_LDS_SCALE_FLOATS floats of LDS, used only with a scale
    template <bool SCALE>
    __device__ __forceinline__ void run(bf16x8* __restrict__ xs_flat, const SkRowScale& sc, float* __restrict__ lds_f) {
        if (!has_work()) return;
        bf16x8(*xs)[XF * 64] = (bf16x8(*)[XF * 64])xs_flat;
        auto xstore = [&](const bf16x8(&src)[XP], int buf) {
#pragma unroll
            for (int p = 0; p < XP; ++p)
                if (XF >= 8 || tid < XF * 64) xs[buf][p * 512 + tid] = src[p];
        };
        f32x16 acc[MT];
#pragma unroll
        for (int i = 0; i < MT; ++i)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][v] = 0.f;

        if constexpr (SCALE) {
            // per-row factor 1 / sqrt(mean(x^2) + eps) from the partial sums of squares, summed in a fixed order:
            // thread (row m, slice s) adds its slice of the parts in ascending order, then the slices in order.
            // The parts lie four to a float4 ([part / 4][row][part % 4]); a thread's loads are issued in batches of
            // eight before any is used (a quad index past the slice re-reads its last quad and adds nothing).
            constexpr int Mp = MT * 32, SL = 512 / Mp;
            const int m = tid % Mp, sl = tid / Mp;
            const int n_q = (sc.n_parts + 3) >> 2, per = (n_q + SL - 1) / SL, q0 = sl * per, q1 = min(q0 + per, n_q);
            const float4* sq = (const float4*)sc.ssq + m;
            float t = 0.f;
            for (int b0 = q0; b0 < q1; b0 += 8) {
                float4 v[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) v[i] = sq[(size_t)min(b0 + i, q1 - 1) * Mp];
#pragma unroll
                for (int i = 0; i < 8; ++i)
                    if (b0 + i < q1) t += (v[i].x + v[i].y) + (v[i].z + v[i].w);
            }
            lds_f[256 + sl * Mp + m] = t;
            __syncthreads();
            if (tid < Mp) {
                float tot = 0.f;
#pragma unroll
                for (int q = 0; q < SL; ++q) tot += lds_f[256 + q * Mp + tid];
                lds_f[tid] = rsqrtf(tot * sc.inv_d + sc.eps);
            }
            // (the barrier below, before the first MFMA, also publishes the factors)
        }

        int nseg = 0;
        xstore(xr[0], 0);
        xload(xr[0], nxt, 0);
        __syncthreads();

        for (;;) {
            const bf16x8* wn = wptr(nxt);
#pragma unroll
            for (int c = 0; c < CPI; ++c) {
#pragma unroll
                for (int j = 0; j < XK; ++j) {
                    const int i = c * XK + j;                         // ring slot (compile-time)
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt) {
                        bf16x8 hi = xs[c & 1][((j * MT + mt) * 2) * 64 + lane];
                        bf16x8 lo = xs[c & 1][((j * MT + mt) * 2 + 1) * 64 + lane];
                        acc[mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(hi, w[i], acc[mt], 0, 0, 0);
                        acc[mt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(lo, w[i], acc[mt], 0, 0, 0);
                    }
                    w[i] = __builtin_nontemporal_load((i < nxt.valid) ? wn + (size_t)i * wstep : zl);
                }
                // the chunk consumed next goes to the other buffer; its register slot is refilled
                // with the chunk one outer iteration further on
                const int nc = (c + 1) % CPI;
                xstore(xr[nc], (c + 1) & 1);
                if (c + 1 < CPI) xload(xr[nc], nxt, c + 1);
                else xload(xr[nc], nx2, 0);
                __syncthreads();
            }
            if (cur.last) {
                // slot = ordinal of this workgroup among those whose ranges meet column group cur.ng: known
                // from the plan for the first segment; every later segment starts its column group
                const int slot = nseg == 0 ? slot0 : 0;
                ++nseg;
                const int nb = cur.ng * 8 + wave;
                if (nb < NB) {
                    // the row stride and the lane's row group are made opaque here so that the row offsets
                    // m * ldo are computed where they are used: hoisted out of the loop (which the compiler
                    // does otherwise) they occupy registers for the whole kernel, 64 of them here and some
                    // 150 in the 128-row kernel
                    int gq = lane >> 5, ldo_here = ldo;
                    asm volatile("" : "+v"(gq), "+s"(ldo_here));
                    float* tile = out + (size_t)__builtin_amdgcn_readfirstlane(slot) * slot_stride;
                    const int col = nb * 32 + (lane & 31);
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt) {
                        const TileStore ts(tile, mt * 32, rows, ldo_here);
#pragma unroll
                        for (int v = 0; v < 16; ++v) {
                            const int m = 8 * (v >> 2) + 4 * gq + (v & 3);
                            float val = acc[mt][v];
                            if constexpr (SCALE) val *= lds_f[mt * 32 + m];
                            ts.put(val, (m * ldo_here + col) * 4);
                        }
                    }
                }
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                    for (int v = 0; v < 16; ++v) acc[mt][v] = 0.f;
            }
            if (nxt.valid == 0) break;
            cur = nxt;
            nxt = nx2;
            nx2 = sk_walk_next<R>(walk, KB);
        }
    }
};
