// Integer stages of the step: arg-max / top-k over the vocabulary, greedy acceptance with
// the fragment cut (paper Section III-B), and the commit of the accepted K/V rows.
#include "sd_internal.h"

#define NEG_INF (-__builtin_inff())

// "better" = larger value, ties to the lower index
static __device__ inline bool better(float v, int i, float bv, int bi) { return v > bv || (v == bv && i < bi); }

static __device__ inline void wave_best(float& v, int& i) {
    for (int o = 32; o > 0; o >>= 1) {
        float ov = __shfl_xor(v, o);
        int oi = __shfl_xor(i, o);
        if (better(ov, oi, v, i)) { v = ov; i = oi; }
    }
}

// ------------------------------------------------------------------------------------------
// Ranking of logit rows straight from the LM head's partial sums, in two stages. Stage 1, one workgroup per (row, chunk of
// the vocabulary): a thread sums the slots of its columns (in slot order), writes the logits out where somebody wants
// them (straight to the caller's dense rows: no padded copy, no second pass), and the workgroup finds the best entry
// (K1: arg-max) or the best k of its chunk. Stage 2: k_verify picks a row's arg-max out of its chunks' by itself; for
// top-k, k_topk_merge. At most 16 chunks, of NPT * 256 ids. One workgroup per row, as before, left most of the
// chip idle (plain decoding: one workgroup, 10 us for the arg-max and 5 + 22 + 5 us for sum, top-10 and copy of four head
// rows, which are 7 + 6 us in this form).
// Top-k of a chunk without rounds over the chunk: the k-th best of the threads' own maxima bounds the chunk's k-th best from
// below, so only entries at or above it (of k threads at most: k * NPT) can belong to the best k; those are listed, and
// an entry's place is the number of better ones. "Better" = larger value, lower id on ties, so places are unique. (k
// rounds of a reduction over the workgroup took 22 us, over single waves 11.5.) Logits of -inf are never picked.
#define RANK_THREADS 256
struct RankOut {
    float* logits;         // NULL, or the summed logits: row r at logits + (map_B ? (r % map_B) * map_H + r / map_B : r) * ld
    int ld, map_B, map_H, vec;      // vec: rows are 16-byte aligned and hold a multiple of four ids
};
// An entry as one 64-bit key: larger key = better (larger value, -0 like +0; lower id on ties); 0 = no entry. Compared as
// (value, id) pairs the counting loops were branches on every entry, 27 us.
static __device__ inline unsigned long long rank_key(float v, int id) {
    const uint32_t u = __float_as_uint(v + 0.f);
    return ((unsigned long long)(u & 0x80000000u ? ~u : u | 0x80000000u) << 32) | (uint32_t)~id;
}
static __device__ inline int key_id(unsigned long long k) { return (int)~(uint32_t)k; }
// how many of list[0..n) are larger than me; the list is in LDS and followed by one free entry if n is odd, which must be 0
static __device__ inline int count_better(const unsigned long long* list, int n, unsigned long long me) {
    int place = 0;
    const ulonglong2* l2 = (const ulonglong2*)list;
#pragma unroll 8
    for (int j = 0; j < (n + 1) / 2; ++j) {
        const ulonglong2 o = l2[j];
        place += (o.x > me) + (o.y > me);
    }
    return place;
}
template <int NPT, bool K1>
__global__ __launch_bounds__(RANK_THREADS) void k_rank_chunks(PartView pv, int row0, int V, int k, RankOut ro,
                                                              void* __restrict__ cand) {
    static_assert(NPT % 4 == 0, "float4 groups");
    const int ch = blockIdx.x, r = blockIdx.y, tid = threadIdx.x;
    [[maybe_unused]] const int wave = tid >> 6, lane = tid & 63;
    const float* row = pv.base + (size_t)(row0 + r) * pv.ld;
    const int c0 = ch * NPT * RANK_THREADS;
    float* out = nullptr;
    if (ro.logits) out = ro.logits + (size_t)(ro.map_B ? (r % ro.map_B) * ro.map_H + r / ro.map_B : r) * ro.ld;
    float v[NPT];
    float bv = NEG_INF;
    int bi = 0x7fffffff;
#pragma unroll
    for (int q = 0; q < NPT / 4; ++q) {
        const int c = c0 + (q * RANK_THREADS + tid) * 4;
        float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
        if (c < V) {                                   // (the partial sums' rows are padded to 32 columns)
            const int n = part_count(pv, c);
#pragma unroll 4
            for (int sp = 0; sp < n; ++sp) {
                const float4 x = *(const float4*)(row + (size_t)sp * pv.slot_stride + c);
                a.x += x.x; a.y += x.y; a.z += x.z; a.w += x.w;
            }
        }
        const float e4[4] = {a.x, a.y, a.z, a.w};
        if (out && c < V) {
            if (ro.vec) *(float4*)(out + c) = a;
            else
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (c + e < V) out[c + e] = e4[e];
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            // ascending ids: the first maximum. (The arg-max of a row of -inf is its first id; top-k never picks a -inf.)
            v[q * 4 + e] = c + e < V ? e4[e] : NEG_INF;
            if (K1 ? c + e < V && better(e4[e], c + e, bv, bi) : v[q * 4 + e] > bv) { bv = v[q * 4 + e]; bi = c + e; }
        }
    }
    if constexpr (K1) {
        __shared__ float2 wbest[RANK_THREADS / 64];
        wave_best(bv, bi);
        if (lane == 0) wbest[wave] = make_float2(bv, __int_as_float(bi));
        __syncthreads();
        if (tid == 0) {
#pragma unroll
            for (int w = 1; w < RANK_THREADS / 64; ++w) {
                const float2 e = wbest[w];
                if (better(e.x, __float_as_int(e.y), bv, bi)) { bv = e.x; bi = __float_as_int(e.y); }
            }
            ((float2*)cand)[(size_t)r * gridDim.x + ch] = make_float2(bv, __int_as_float(bi));
        }
    } else {
        __shared__ __attribute__((aligned(16))) unsigned long long own[RANK_THREADS];      // the threads' maxima
        __shared__ __attribute__((aligned(16))) unsigned long long lst[32 * NPT + 2];      // k <= 32
        __shared__ unsigned long long bound;
        __shared__ int count;
        const unsigned long long mine = bi == 0x7fffffff ? 0ull : rank_key(bv, bi);
        own[tid] = mine;
        if (tid == 0) { count = 0; bound = 0ull; }
        __syncthreads();
        // (fewer than k threads with an entry: no bound, every entry is listed)
        if (mine && count_better(own, RANK_THREADS, mine) == k - 1) bound = mine;
        __syncthreads();
        const unsigned long long least = bound;
        if (mine >= least && mine) {
#pragma unroll
            for (int j = 0; j < NPT; ++j) {
                const int c = c0 + ((j >> 2) * RANK_THREADS + tid) * 4 + (j & 3);
                const unsigned long long e = rank_key(v[j], c);
                if (v[j] > NEG_INF && e >= least) lst[atomicAdd(&count, 1)] = e;
            }
        }
        __syncthreads();
        const int n = count;
        if (tid == 0) lst[n] = 0ull;                       // (an odd list is read in pairs)
        __syncthreads();
        unsigned long long* out_k = (unsigned long long*)cand + ((size_t)r * gridDim.x + ch) * k;
        for (int e = tid; e < n; e += RANK_THREADS) {
            const int place = count_better(lst, n, lst[e]);
            if (place < k) out_k[place] = lst[e];
        }
        for (int e = n + tid; e < k; e += RANK_THREADS) out_k[e] = 0ull;           // a chunk of fewer than k
    }
}

// the best k of a row's n = chunks * k entries, by the same counting; row r = head i * B + b of the pass
__global__ __launch_bounds__(RANK_THREADS) void k_topk_merge(const unsigned long long* __restrict__ cand, int n, int k,
                                                             int32_t* __restrict__ out, int B, int H, SeqList sl) {
    extern __shared__ __attribute__((aligned(16))) unsigned long long all[];       // n + 2 entries
    __shared__ int found;
    const int r = blockIdx.x, i = r / B, b = r % B, tid = threadIdx.x;
    if (tid == 0) { found = 0; all[n] = 0ull; }
    for (int j = tid; j < n; j += RANK_THREADS) all[j] = cand[(size_t)r * n + j];
    __syncthreads();
    int32_t* o = out + ((size_t)sl.seq[b] * H + i) * k;
    for (int e = tid; e < n; e += RANK_THREADS) {
        const unsigned long long me = all[e];
        if (!me) continue;                             // a chunk of fewer than k
        const int place = count_better(all, n, me);
        if (place < k) { o[place] = key_id(me); atomicAdd(&found, 1); }
    }
    __syncthreads();
    for (int e = found + tid; e < k; e += RANK_THREADS) o[e] = 0x7fffffff;      // a row of fewer than k finite logits
}

int rank_chunks(int V) {
    const int npt = V <= 32768 ? 8 : V <= 65536 ? 16 : 40;         // 40: 163840 ids, the most a model may have
    return (V + npt * RANK_THREADS - 1) / (npt * RANK_THREADS);
}
static RankOut rank_out(float* logits, int ld, int V, int map_B, int map_H) {
    return RankOut{logits, ld, map_B, map_H, (((uintptr_t)logits & 15) == 0 && ld % 4 == 0 && V % 4 == 0) ? 1 : 0};
}
#define RANK(K1_, k_)                                                                                                    \
    do {                                                                                                                 \
        const dim3 grid(rank_chunks(V), rows);                                                                           \
        if (V <= 32768) hipLaunchKernelGGL((k_rank_chunks<8, K1_>), grid, dim3(RANK_THREADS), 0, s, pv, row0, V, k_, ro, cand);  \
        else if (V <= 65536) hipLaunchKernelGGL((k_rank_chunks<16, K1_>), grid, dim3(RANK_THREADS), 0, s, pv, row0, V, k_, ro, cand); \
        else hipLaunchKernelGGL((k_rank_chunks<40, K1_>), grid, dim3(RANK_THREADS), 0, s, pv, row0, V, k_, ro, cand);    \
    } while (0)
void launch_rank_best(PartView pv, int row0, int rows, int V, float* logits, int ld, float2* cand, hipStream_t s) {
    const RankOut ro = rank_out(logits, ld, V, 0, 0);
    RANK(true, 1);
}
void launch_topk(PartView pv, int row0, int V, int k, int32_t* out, int B, int H, const SeqList& sl, float* head_logits,
                 void* cand, hipStream_t s) {
    const int rows = B * H, n = rank_chunks(V) * k;
    const RankOut ro = rank_out(head_logits, V, V, B, H);
    RANK(false, k);
    hipLaunchKernelGGL(k_topk_merge, dim3(rows), dim3(RANK_THREADS), (size_t)(n + 2) * 8, s, (const unsigned long long*)cand, n, k, out, B, H, sl);
}
#undef RANK

// a row's arg-max out of its chunks' best entries (chunks in ascending ids: the first maximum)
static __device__ inline int best_of_chunks(const float2* __restrict__ best, int nch) {
    float2 e[16];                                      // (16 chunks at most; past the last: the last again)
#pragma unroll
    for (int c = 0; c < 16; ++c) e[c] = best[min(c, nch - 1)];
    float bv = e[0].x;
    int bi = __float_as_int(e[0].y);
#pragma unroll
    for (int c = 1; c < 16; ++c)
        if (better(e[c].x, __float_as_int(e[c].y), bv, bi)) { bv = e[c].x; bi = __float_as_int(e[c].y); }
    return bi;
}

// ------------------------------------------------------------------------------------------
// Sampling decoding, statistics of the base distribution of every tree row at a temperature:
// with x_v = (logit_v - max) / temperature, Z = sum exp(x_v), E = sum exp(x_v) x_v, the entropy
// of softmax is H = log Z - E / Z and the typical-acceptance threshold is min(eps, delta exp(-H)).
// A token passes iff exp(x_tok) / Z > threshold, i.e. x_tok > c with
// c = min(log eps, log delta - H) + log Z. One workgroup of 1024 threads per row, the row kept
// in registers between the two reductions; thread sums in fp32, cross-thread sums in fp64.
#define RS_THREADS 1024
static __device__ inline double block_sum_f64(double v, double* sh) {
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    __syncthreads();                                   // sh may still be read from the previous call
    if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
    __syncthreads();
    double t = 0.0;
    for (int w = 0; w < RS_THREADS / 64; ++w) t += sh[w];
    return t;
}
template <int NPT>
__global__ __launch_bounds__(RS_THREADS) void k_row_stats(const float* __restrict__ logits, int ld, int V,
                                                          float4* __restrict__ stats, int T, int Tp,
                                                          float inv_temperature, float log_eps, float log_delta) {
    const int j = blockIdx.x, b = blockIdx.y, tid = threadIdx.x;
    const size_t r = (size_t)b * Tp + j;
    const float* row = logits + r * ld;
    float v[NPT];
    float mx = NEG_INF;
#pragma unroll
    for (int i = 0; i < NPT; ++i) {
        const int c = i * RS_THREADS + tid;
        v[i] = c < V ? row[c] : NEG_INF;
        mx = fmaxf(mx, v[i]);
    }
    __shared__ float smax[RS_THREADS / 64];
    __shared__ double ssum[RS_THREADS / 64];
    for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
    if ((tid & 63) == 0) smax[tid >> 6] = mx;
    __syncthreads();
    mx = smax[0];
    for (int w = 1; w < RS_THREADS / 64; ++w) mx = fmaxf(mx, smax[w]);
    float z = 0.f, e = 0.f;
#pragma unroll
    for (int i = 0; i < NPT; ++i) {
        const int c = i * RS_THREADS + tid;
        if (c < V) {
            const float x = (v[i] - mx) * inv_temperature;
            const float ex = __expf(x);
            z += ex;
            e += ex * x;                               // exp(x) x -> 0 as x -> -inf
        }
    }
    const double Z = block_sum_f64((double)z, ssum);
    const double E = block_sum_f64((double)e, ssum);
    if (tid == 0) {
        const double H = log(Z) - E / Z;
        const double log_thr = fmin((double)log_eps, (double)log_delta - H);
        stats[r] = make_float4(mx, (float)Z, (float)H, (float)(log_thr + log(Z)));
    }
}

void launch_row_stats(const float* logits, int ld, int V, float4* stats, int B, int T, int Tp, float inv_temperature,
                      float epsilon, float delta, hipStream_t s) {
    const float log_eps = epsilon > 0.f ? logf(epsilon) : NEG_INF, log_delta = delta > 0.f ? logf(delta) : NEG_INF;
    const int npt = (V + RS_THREADS - 1) / RS_THREADS;
#define RS(N) hipLaunchKernelGGL((k_row_stats<N>), dim3(T, B), dim3(RS_THREADS), 0, s, logits, ld, V, stats, T, Tp, \
                                 inv_temperature, log_eps, log_delta)
    if (npt <= 1) RS(1);
    else if (npt <= 4) RS(4);
    else if (npt <= 16) RS(16);
    else if (npt <= 32) RS(32);
    else if (npt <= 64) RS(64);
    else RS(160);
#undef RS
}

// ------------------------------------------------------------------------------------------
// Sampling decoding, the next root: the smallest token id whose cumulative probability under
// softmax(logits[last_row] / temperature) exceeds u. One workgroup of 16 waves per sequence.
// Wave w owns the contiguous ids [w*S, (w+1)*S), lane l of group j the id w*S + 64 j + l: the
// maximum, then the weights exp((l - max)/temp). The weights of the segment that holds the target u * total go to
// LDS, where every lane sums a whole group of 64 in id order; one scan over the groups and one inside the group found
// give the id. (Walking the segment group by group, a scan each, took 22 us at 32 k ids; this form 8.) Sums are in fp64,
// so the draw only differs from an exact one when u lies within fp32 rounding of the weights of a boundary of the CDF.
static __device__ inline double wave_incl_scan_f64(double v, int lane) {
    for (int o = 1; o < 64; o <<= 1) {
        double t = __shfl_up(v, o);
        if (lane >= o) v += t;
    }
    return v;
}
// NPT: groups of a wave, at most. KEEP: the weights stay in registers, up to 65536 ids (64 of them per lane: 14 registers
// spill, and reading the row twice is slower all the same: 12.6 against 15.1 us at 65536 ids, level at 33000); beyond, where 160 would spill 237
// registers, the row is read again from the caches for the sum, sixteen groups' loads in flight, and all waves fetch the
// segment that holds the target, so that no wave is left alone with it. One row / eight rows of 100000, 128256 and
// 163840 ids: 23 / 24, 26 / 27, 32 / 32 us; spilled 42 / 43, 45 / 46, 47 / 47; walking the segment a scan per 64 ids
// 26 / 50, 35 / 65, 74 / 80 (the longer, the further into its segment the draw falls).
template <int NPT, bool KEEP>
__global__ __launch_bounds__(RS_THREADS) void k_sample_root(const float* __restrict__ logits, int ld, int V,
                                                            const int32_t* __restrict__ last_row,
                                                            const float* __restrict__ u, float inv_temperature,
                                                            int32_t* __restrict__ root_tok, int n_rows) {
    constexpr int NW = RS_THREADS / 64;
    const int b = blockIdx.x, tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
    const int r = last_row[b];
    if (r < 0 || r >= n_rows) {                        // uniform over the workgroup
        if (tid == 0) root_tok[b] = -1;
        return;
    }
    const float* row = logits + (size_t)r * ld;
    __shared__ float smax[NW];
    __shared__ double wsum[NW];
    __shared__ float ws[NPT * 65];                     // one segment's weights, [group][64 + 1]
    const int S = ((V + NW - 1) / NW + 63) & ~63;      // segment length, a multiple of the wave size
    int s0 = min(wave * S, V), s1 = min(s0 + S, V);
    constexpr int U = KEEP ? NPT : 16;                 // groups whose loads are issued together
    int groups = (s1 - s0 + 63) / 64;
    float v[U];
    auto load = [&](int j0) {                          // groups j0 .. j0 + U - 1 of this wave's segment
#pragma unroll
        for (int j = 0; j < U; ++j) {
            const int c = s0 + (j0 + j) * 64 + lane;
            if constexpr (KEEP) v[j] = c < s1 ? row[c] : NEG_INF;
            else v[j] = row[min(c, V - 1)];
        }
    };
    float mx = NEG_INF;
    for (int j0 = 0; j0 < (KEEP ? 1 : groups); j0 += U) {
        load(j0);
#pragma unroll
        for (int j = 0; j < U; ++j) mx = fmaxf(mx, KEEP || s0 + (j0 + j) * 64 + lane < s1 ? v[j] : NEG_INF);
    }
    for (int o = 32; o > 0; o >>= 1) mx = fmaxf(mx, __shfl_xor(mx, o));
    if (lane == 0) smax[wave] = mx;
    __syncthreads();
    mx = smax[0];
    for (int w = 1; w < NW; ++w) mx = fmaxf(mx, smax[w]);
    auto weight = [&](int j0, int j) { return s0 + (j0 + j) * 64 + lane < s1 ? __expf((v[j] - mx) * inv_temperature) : 0.f; };
    double part = 0.0;
    for (int j0 = 0; j0 < (KEEP ? 1 : groups); j0 += U) {
        if constexpr (!KEEP) load(j0);
#pragma unroll
        for (int j = 0; j < U; ++j) {
            v[j] = weight(j0, j);
            part += (double)v[j];
        }
    }
    for (int o = 32; o > 0; o >>= 1) part += __shfl_xor(part, o);
    if (lane == 0) wsum[wave] = part;
    __syncthreads();
    double total = 0.0;
    for (int w = 0; w < NW; ++w) total += wsum[w];
    const double target = (double)u[b] * total;
    // the segment that holds the target; if rounding leaves none, the last one that has any mass, taken to its end
    int seg = -1, last_mass = 0;
    double base = 0.0, acc = 0.0;
    for (int w = 0; w < NW; ++w) {
        if (wsum[w] > 0.0) last_mass = w;
        if (seg < 0 && acc + wsum[w] > target) { seg = w; base = acc; }
        acc += wsum[w];
    }
    const bool to_end = seg < 0;
    if (to_end) seg = last_mass;
    int last_pos;                                      // the last id with mass
    if constexpr (KEEP) {
        if (wave != seg) return;                       // (the rest is this wave's alone: no barrier follows)
        last_pos = s0;
#pragma unroll
        for (int j = 0; j < NPT; ++j) {
            ws[j * 65 + lane] = v[j];
            const unsigned long long pos = __ballot(v[j] > 0.f);
            if (pos) last_pos = s0 + j * 64 + 63 - __builtin_clzll(pos);
        }
        __builtin_amdgcn_wave_barrier();
    } else {
        // every wave fetches its share of that segment's groups; the draw is the first wave's
        __shared__ int last;
        s0 = min(seg * S, V);
        s1 = min(s0 + S, V);
        groups = (s1 - s0 + 63) / 64;
        if (tid == 0) last = s0;
        __syncthreads();
        float x[NPT / NW];
#pragma unroll
        for (int i = 0; i < NPT / NW; ++i) x[i] = row[min(s0 + (wave + i * NW) * 64 + lane, V - 1)];
#pragma unroll
        for (int i = 0; i < NPT / NW; ++i) {
            const int g = wave + i * NW, c = s0 + g * 64 + lane;
            const float e = c < s1 ? __expf((x[i] - mx) * inv_temperature) : 0.f;
            if (g < groups) ws[g * 65 + lane] = e;
            const unsigned long long pos = __ballot(e > 0.f);
            if (pos && lane == 0) atomicMax(&last, s0 + g * 64 + 63 - __builtin_clzll(pos));
        }
        __syncthreads();
        if (wave != 0) return;
        last_pos = last;
    }
    int pick = -1;
    for (int g0 = 0; g0 < groups && pick < 0 && !to_end; g0 += 64) {
        double gsum = 0.0;
        if (g0 + lane < groups)
#pragma unroll 16
            for (int i = 0; i < 64; ++i) gsum += (double)ws[(g0 + lane) * 65 + i];
        const double cum = base + wave_incl_scan_f64(gsum, lane);
        // (a group without mass is never the one: its place in the scan can round past the target that the sum before it,
        // the same number exactly, does not pass)
        const unsigned long long hit = __ballot(gsum > 0.0 && cum > target);
        if (hit) {
            const int gl = __builtin_ctzll(hit), g = g0 + gl;
            const double before = gl ? __shfl(cum, gl - 1) : base;
            const double e = (double)ws[g * 65 + lane];
            const unsigned long long in = __ballot(e > 0.0 && before + wave_incl_scan_f64(e, lane) > target);
            const unsigned long long mass = __ballot(e > 0.0);
            // (the two sums of a group may differ in the last bit: then its last id with mass)
            pick = s0 + g * 64 + (in ? __builtin_ctzll(in) : 63 - __builtin_clzll(mass));
        }
        base = __shfl(cum, 63);
    }
    if (lane == 0) root_tok[b] = pick >= 0 ? pick : last_pos;
}

void launch_sample_root(const float* logits, int ld, int V, const int32_t* last_row, const float* u,
                        float inv_temperature, int32_t* root_tok, int B, int n_rows, hipStream_t s) {
    const int npt = (((V + RS_THREADS / 64 - 1) / (RS_THREADS / 64) + 63) & ~63) / 64;
#define SR(N, KEEP_) hipLaunchKernelGGL((k_sample_root<N, KEEP_>), dim3(B), dim3(RS_THREADS), 0, s, logits, ld, V, last_row, u, \
                                        inv_temperature, root_tok, n_rows)
    if (npt <= 4) SR(4, true);
    else if (npt <= 16) SR(16, true);
    else if (npt <= 32) SR(32, true);
    else if (npt <= 64) SR(64, true);
    else SR(160, false);                               // 163840 ids
#undef SR
}

// ------------------------------------------------------------------------------------------
// Greedy acceptance + fragment cut. One workgroup of 64*NW >= T threads per sequence, thread
// j = tree node j (NW = 2 for trees of up to 128 nodes, 4 beyond).
//   match[j]  = tok[j] == am[parent[j]]                     (root: true); under sampling decoding
//               instead: p(tok[j] | parent) > min(eps, delta * exp(-entropy)), from k_row_stats
//   ok[j]     = match holds on every node of j's root path  (prefix-closed acceptance): with
//               the per-wave ballots of `match` gathered into a T-bit mask, ok[j] is one
//               AND of j's ancestor bitset with the complement of that mask
//   best      = deepest ok node (lowest index on equal depth), by wavefront reduction
//   chain     = best's ancestor bitset; node j of the chain sits at chain index depth[j]
//   cut       = 1 + largest chain index whose token is in the stop set; without any stop
//               token: whole chain (keep_all) or 1 (keep_one)
template <int NW>
__global__ __launch_bounds__(64 * NW) void k_verify(VerifyArgs a) {
    const int b = blockIdx.x, j = threadIdx.x, T = a.T, H = a.H;
    const bool valid = j < T;
    const int32_t* tok = a.tok + (size_t)b * a.src_stride;
    __shared__ unsigned long long matchw[NW], bestanc[NW];
    __shared__ int wkey[NW], stopmax[NW], am_s[64 * NW];
    // the base arg-max of every node: given, or picked out of the chunks' best entries (k_rank_chunks)
    int amj = 0;
    if (valid) {
        const size_t r = (size_t)b * a.src_stride + j;
        amj = a.best ? best_of_chunks(a.best + r * a.n_chunks, a.n_chunks) : a.am[r];
        if (a.am_out) a.am_out[(size_t)b * T + j] = amj;
    }
    am_s[j] = amj;
    __syncthreads();
    int dj = 0, tj = 0, pj = -1;
    unsigned long long anc[NW] = {};
    bool match = false;
    if (valid) {
        dj = a.depth[j];
        pj = a.parent[j];
        tj = tok[j];
        if (j == 0) {
            match = true;
        } else if (a.row_stats) {
            // the base model's probability of this token at its parent exceeds the threshold of that
            // row, tested on the log side: (logit - max) / temperature > log(threshold * Z)
            const size_t r = (size_t)b * a.src_stride + pj;
            const float4 st = a.row_stats[r];
            match = false;
            if (tj >= 0 && tj < a.V) match = (a.logits[r * a.ld + tj] - st.x) * a.inv_temperature > st.w;
        } else {
            match = tj == am_s[pj];
        }
        for (int i = j, guard = 0; i >= 0 && guard <= H; i = a.parent[i], ++guard) anc[i >> 6] |= 1ull << (i & 63);
    }
    unsigned long long bal = __ballot(match);
    if ((j & 63) == 0) matchw[j >> 6] = bal;
    __syncthreads();
    unsigned long long miss = 0ull;
#pragma unroll
    for (int w = 0; w < NW; ++w) miss |= anc[w] & ~matchw[w];
    const bool ok = valid && miss == 0ull;
    // deepest accepted node, lowest index on ties: maximise depth * 256 + (255 - j)
    static_assert(SD_MAX_TREE <= 256, "the key holds the node index in 8 bits");
    int key = ok ? dj * 256 + (255 - j) : -1;
    for (int o = 32; o > 0; o >>= 1) key = max(key, __shfl_xor(key, o));
    if ((j & 63) == 0) wkey[j >> 6] = key;
    __syncthreads();
    key = wkey[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) key = max(key, wkey[w]);
    const int best = 255 - (key & 255);
    const int n_raw = (key >> 8) + 1;
    if (j == best) {
#pragma unroll
        for (int w = 0; w < NW; ++w) bestanc[w] = anc[w];
    }
    __syncthreads();
    const bool on_chain = valid && ((bestanc[j >> 6] >> (j & 63)) & 1ull);
    const bool is_stop = on_chain && tj >= 0 && tj < a.V && ((a.stop_mask[tj >> 5] >> (tj & 31)) & 1u);
    int sm = is_stop ? dj : -1;
    for (int o = 32; o > 0; o >>= 1) sm = max(sm, __shfl_xor(sm, o));
    if ((j & 63) == 0) stopmax[j >> 6] = sm;
    __syncthreads();
    sm = stopmax[0];
#pragma unroll
    for (int w = 1; w < NW; ++w) sm = max(sm, stopmax[w]);
    const int n_acc = sm >= 0 ? sm + 1 : (a.fallback == SD_TRUNC_KEEP_ALL ? n_raw : 1);
    const int W = H + 1;
    if (on_chain && dj < n_acc) {
        a.tokens[(size_t)b * W + dj] = tj;
        a.src_slots[(size_t)b * W + dj] = j;
        if (dj == n_acc - 1) {
            if (a.root_tok) a.root_tok[b] = amj;
            if (a.last_row) a.last_row[b] = b * a.Tp + j;
        }
    }
    if (j >= n_acc && j < W) {
        a.tokens[(size_t)b * W + j] = -1;
        a.src_slots[(size_t)b * W + j] = -1;
    }
    if (j == 0) {
        a.n_accept[b] = n_acc;
        if (a.n_accept_raw) a.n_accept_raw[b] = n_raw;
        if (a.kv_len) {
            int n = a.kv_len[b];
            a.n_old[b] = n;
            a.kv_len[b] = n + n_acc;
        }
    }
}

void launch_verify(const VerifyArgs& a, int B, hipStream_t s) {
    if (a.T <= 128) hipLaunchKernelGGL(k_verify<2>, dim3(B), dim3(128), 0, s, a);
    else hipLaunchKernelGGL(k_verify<4>, dim3(B), dim3(256), 0, s, a);
}

// ------------------------------------------------------------------------------------------
// Commit the kept nodes' K/V rows: tree-scratch row src_slots[j] -> cache row n_old + j, for
// every layer and head. A kept node at chain index j was rotated for position n_old + j
// already (depth = chain index), so this is a pure copy.
// grid: x = head, y = sequence b of the pass that filled the scratch (sequence rm.seq[b] of the cache; rm.off[b] = entry of
// src_slots, n_accept and n_old + 256 * its last scratch row, which a slot past it stands for), z = layer; eight waves
// that share a list of wave-sized tasks, every task a run of whole 16-byte pieces that lie side by side in the cache:
//   values: a 16-byte piece of the value layout holds one dim of EIGHT rows (a "group": of a 16-row half of a block,
//     the four rows of one quad and of the quad two further on), so a row cannot move as a piece, and a piece
//     written in parts (2-byte elements, or its 8-byte halves from two workgroups) leaves the memory partial lines.
//     One task = one half x 32 dims: a lane owns one piece, reads it unless all of its eight rows are replaced
//     (its other rows are committed rows, which must survive, or rows past the new length, which nobody reads), takes
//     the new rows' elements and writes the piece whole: 1 KiB per wave, in order (writing only the 8-byte half that
//     has new rows, where one does not, was measured and is slower, short lists included). The new rows' elements
//     come from a copy in LDS of the scratch groups that hold a kept row, fetched once as whole pieces: picked out
//     of global memory two bytes at a time they cost a cache lookup per element and lane, eight times the lookups
//     of everything else here (MIRROR = false: no room for that copy, the elements are gathered from global
//     memory).
//   keys: a row's 16-byte pieces move as they are; one task = 8 rows x 8 pieces, rows fastest (the same piece of
//     neighbouring rows is 16 bytes further on, so eight lanes write 128 contiguous bytes).
// Every piece has one owner, and only this workgroup touches this layer's blocks of its (sequence, head).
#define KVC_THREADS 512
typedef uint16_t u16x8 __attribute__((ext_vector_type(8)));
static __device__ inline int vgroup_of(int c) { return (c >> 5) * 4 + ((c >> 4) & 1) * 2 + ((c >> 2) & 1); }
template <bool MIRROR>
__global__ __launch_bounds__(KVC_THREADS) void k_kv_commit(
    const uint16_t* __restrict__ kt, const uint16_t* __restrict__ vt, uint16_t* __restrict__ kc,
    uint16_t* __restrict__ vc, const int32_t* __restrict__ src_slots, const int32_t* __restrict__ n_accept,
    const int32_t* __restrict__ n_old, RowMap rm, int nh, int hd, int TB, int cap_blocks, int W, int L, int lpw,
    size_t layer_stride_t, size_t layer_stride_c) {
    extern __shared__ __align__(16) uint16_t kvc_mirror[];          // [kept group][hd / 32][32 dims][8 rows]
    __shared__ int s_slots[SD_MAX_TREE];
    __shared__ uint32_t s_need;
    const int h = blockIdx.x, b = blockIdx.y, tid = threadIdx.x;
    const int l0 = blockIdx.z * lpw, l1 = min(l0 + lpw, L);
    const int wave = tid >> 6, lane = tid & 63;
    const int lst = rm.off[b] & 255, last = rm.off[b] >> 8;         // whose list, count and old length these are; its last row
    const int a = min(n_accept[lst], W);                            // <= SD_MAX_TREE < KVC_THREADS
    if (a <= 0) return;
    const int n = n_old[lst];
    const int slot = tid < a ? min(max(src_slots[(size_t)lst * W + tid], 0), last) : 0;
    if (tid == 0) s_need = 0;
    __syncthreads();
    if (tid < a) {
        s_slots[tid] = slot;
        if constexpr (MIRROR) atomicOr(&s_need, 1u << vgroup_of(slot));
    }
    __syncthreads();
    const size_t toff0 = ((size_t)b * nh + h) * TB * (32 * hd);
    const size_t coff0 = ((size_t)rm.seq[b] * nh + h) * cap_blocks * (32 * hd);
    const int EB = hd / 32, KP = hd / 64;                  // wave tasks per 16-row half (values), per 8 rows (keys)
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    const uint32_t need = s_need;
    const int half0 = n >> 4, nV = (((n + a - 1) >> 4) - half0 + 1) * EB;
    const int NT = nV + ((a + 7) >> 3) * KP;
    // The counts, the slots and the set of groups are the same for every layer: a workgroup reads them once and
    // then goes through its layers (the same number of times for every wave: all of them reach the barriers).
    for (int l = l0; l < l1; ++l) {
        const size_t toff = l * layer_stride_t + toff0, coff = l * layer_stride_c + coff0;
        if constexpr (MIRROR) {                            // (the launch has room for min(W, groups of the scratch) groups)
            if (l > l0) __syncthreads();                   // the previous layer's readers are done
            for (int i = tid; i < TB * 4 * EB * 32; i += KVC_THREADS) {
                const int grp = i / (EB * 32), eb = (i >> 5) % EB, er = i & 31;
                if ((need >> grp) & 1u) {
                    const int c = (grp >> 2) * 32 + ((grp >> 1) & 1) * 16 + (grp & 1) * 4;   // the group's first row
                    const int at = ((__popc(need & ((1u << grp) - 1u)) * EB + eb) * 32 + er) * 8;
                    *(u16x8*)(kvc_mirror + at) = *(const u16x8*)(vt + toff + vblk_index(c, eb * 32 + er, hd));
                }
            }
            __syncthreads();
        }
        for (int tl = wave; tl < NT; tl += KVC_THREADS / 64) {
            if (tl < nV) {
                const int eb = tl % EB, er = lane & 31, e = eb * 32 + er;
                const int row0 = (half0 + tl / EB) * 16 + (lane >> 5) * 4;   // the piece's rows: row0 + {0..3, 8..11}
                const int lo = n - row0, hi = n + a - row0;                   // new rows: offsets lo <= r < hi
                const bool any = (lo < 4 && hi > 0) || (lo < 12 && hi > 8);
                const bool full = lo <= 0 && hi >= 12;
                if (!any) continue;
                uint16_t* piece = vc + coff + vblk_index(row0, e, hd);
                u16x8 v = {0, 0, 0, 0, 0, 0, 0, 0}, g;
                if (!full) v = *(const u16x8*)piece;
#pragma unroll
                for (int q = 0; q < 8; ++q) {              // (any kept row's element where the piece's row stays)
                    const int c = s_slots[min(max((q >> 2) * 8 + (q & 3) - lo, 0), a - 1)];
                    if constexpr (MIRROR) {
                        const int cs = __popc(need & ((1u << vgroup_of(c)) - 1u));
                        g[q] = kvc_mirror[((cs * EB + eb) * 32 + er) * 8 + ((c >> 3) & 1) * 4 + (c & 3)];
                    } else {
                        g[q] = vt[toff + vblk_index(c, e, hd)];
                    }
                }
#pragma unroll
                for (int q = 0; q < 8; ++q) {
                    const int r = (q >> 2) * 8 + (q & 3);
                    if (r >= lo && r < hi) v[q] = g[q];
                }
                *(u16x8*)piece = v;
            } else {
                const int tk = tl - nV;
                const int j = (tk / KP) * 8 + (lane & 7), e = ((tk % KP) * 8 + (lane >> 3)) * 8;
                if (j < a)
                    *(u32x4*)(kc + coff + kblk_index(n + j, e, hd)) =
                        *(const u32x4*)(kt + toff + kblk_index(s_slots[j], e, hd));
            }
        }
    }
}

void launch_kv_commit(const void* kt_all, const void* vt_all, void* kc_all, void* vc_all, const int32_t* src_slots,
                      const int32_t* n_accept, const int32_t* n_old, const RowMap& rm, int kv_B, int L, int B, int nh, int hd,
                      int TB, int cap_blocks, int W, hipStream_t s) {
    size_t lst = (size_t)B * nh * TB * 32 * hd, lsc = (size_t)kv_B * nh * cap_blocks * 32 * hd;
    // LDS copy of the scratch groups (8 rows x hd) with a kept row: at most one per row, at most all of them
    const int groups = W < TB * 4 ? W : TB * 4;
    const size_t mirror = (size_t)groups * 8 * hd * 2;
    int lpw = (int)((size_t)B * nh * L / 1024);            // layers per workgroup: one while the launch is small
    lpw = lpw < 1 ? 1 : lpw > L ? L : lpw;
#define KVC(MIRROR_, lds_)                                                                                                  \
    hipLaunchKernelGGL(k_kv_commit<MIRROR_>, dim3(nh, B, (L + lpw - 1) / lpw), dim3(KVC_THREADS), lds_, s,                 \
                       (const uint16_t*)kt_all, (const uint16_t*)vt_all, (uint16_t*)kc_all, (uint16_t*)vc_all, src_slots,  \
                       n_accept, n_old, rm, nh, hd, TB, cap_blocks, W, L, lpw, lst, lsc)
    if (mirror <= 60 * 1024) KVC(true, mirror);
    else KVC(false, 0);                                    // (eight-block scratch at head_dim 128, 31 rows or more)
#undef KVC
}

// ------------------------------------------------------------------------------------------
// Natural-layout rows [nrows][nh][hd] <-> one sequence's cache blocks of one layer: bytes moved once, so a workgroup owns
// one 32-row block of one head and everything moves in 16-byte pieces. Keys keep their pieces (a row's eight dims), eight
// lanes on neighbouring rows, so that both sides are whole 128-byte runs; a value piece holds one dim of eight rows, so
// the block is turned through LDS, and a piece some of whose rows are not asked for is read, patched and written back
// by its one owner. (One thread per element and two-byte accesses took 17.8 us for 1003 rows at the 7B shape, 1.8 TB/s;
// this form 8 us.) VEC: the caller's arrays are 16-byte aligned; else they are read and written by elements.
template <bool VEC>
static __device__ __forceinline__ u16x8 load_piece(const uint16_t* p) {
    if constexpr (VEC) return *(const u16x8*)p;
    u16x8 v;
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = p[i];
    return v;
}
template <bool VEC>
static __device__ __forceinline__ void store_piece(uint16_t* p, const u16x8& v) {
    if constexpr (VEC) { *(u16x8*)p = v; return; }
#pragma unroll
    for (int i = 0; i < 8; ++i) p[i] = v[i];
}
template <int HD, bool TO_CACHE, bool VEC>
__global__ __launch_bounds__(256) void k_kv_rows(uint16_t* __restrict__ kc, uint16_t* __restrict__ vc, uint16_t* __restrict__ k_rows,
                                                 uint16_t* __restrict__ v_rows, int row0, int nrows, int nh, int cap_blocks) {
    constexpr int PC = HD / 8;                         // pieces of a row
    __shared__ __attribute__((aligned(16))) uint16_t tile[32][HD + 8];
    const int blk = (row0 >> 5) + blockIdx.x, h = blockIdx.y, tid = threadIdx.x;
    const size_t hoff = (size_t)h * cap_blocks * (32 * HD);
    const int first = blk * 32 - row0;                 // natural row of the block's row 0 (negative: before the range)
    auto nat = [&](int r) { return ((size_t)(first + r) * nh + h) * HD; };
    auto asked = [&](int r) { return first + r >= 0 && first + r < nrows; };
    if constexpr (TO_CACHE) {                          // values of the rows asked for -> LDS
        for (int i = tid; i < 32 * PC; i += 256) {
            const int r = i / PC, e = (i % PC) * 8;
            if (asked(r)) *(u16x8*)&tile[r][e] = load_piece<VEC>(v_rows + nat(r) + e);
        }
    }
    for (int i = tid; i < 32 * PC; i += 256) {         // keys: eight rows x eight pieces per wave
        const int r = ((i >> 6) & 3) * 8 + (i & 7), e = ((i >> 8) * 8 + ((i >> 3) & 7)) * 8;
        if (!asked(r)) continue;
        uint16_t* c = kc + hoff + kblk_index(blk * 32 + r, e, HD);
        if constexpr (TO_CACHE) *(u16x8*)c = load_piece<VEC>(k_rows + nat(r) + e);
        else store_piece<VEC>(k_rows + nat(r) + e, *(const u16x8*)c);
    }
    if constexpr (TO_CACHE) __syncthreads();
    for (int i = tid; i < 32 * PC; i += 256) {         // value pieces in cache order: half, 32-dim block, quad, dim
        const int er = i & 31, g = (i >> 5) & 1, eb = (i >> 6) % (HD / 32), p = (i >> 6) / (HD / 32), e = eb * 32 + er;
        const int r0 = p * 16 + g * 4;                 // the piece's rows: r0 + {0..3, 8..11}
        uint16_t* c = vc + hoff + vblk_index(blk * 32 + r0, e, HD);
        bool any = false, all = true;
#pragma unroll
        for (int q = 0; q < 8; ++q) { const bool a = asked(r0 + (q >> 2) * 8 + (q & 3)); any |= a; all &= a; }
        if (!any) continue;
        u16x8 v = {0, 0, 0, 0, 0, 0, 0, 0};
        if (!TO_CACHE || !all) v = *(const u16x8*)c;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int r = r0 + (q >> 2) * 8 + (q & 3);
            if constexpr (TO_CACHE) { if (asked(r)) v[q] = tile[r][e]; }
            else tile[r][e] = v[q];
        }
        if constexpr (TO_CACHE) *(u16x8*)c = v;
    }
    if constexpr (!TO_CACHE) {
        __syncthreads();
        for (int i = tid; i < 32 * PC; i += 256) {
            const int r = i / PC, e = (i % PC) * 8;
            if (asked(r)) store_piece<VEC>(v_rows + nat(r) + e, *(const u16x8*)&tile[r][e]);
        }
    }
}

void launch_kv_rows(void* kc, void* vc, void* k_rows, void* v_rows, int row0, int nrows, int nh, int hd,
                    int cap_blocks, int to_cache, hipStream_t s) {
    const dim3 grid((row0 + nrows - 1) / 32 - row0 / 32 + 1, nh);
    const bool vec = ((((uintptr_t)k_rows) | ((uintptr_t)v_rows)) & 15) == 0;
#define KV_ROWS(HD_, TO_, VEC_)                                                                                        \
    hipLaunchKernelGGL((k_kv_rows<HD_, TO_, VEC_>), grid, dim3(256), 0, s, (uint16_t*)kc, (uint16_t*)vc,              \
                       (uint16_t*)k_rows, (uint16_t*)v_rows, row0, nrows, nh, cap_blocks)
#define KV_ROWS2(HD_, TO_) do { if (vec) KV_ROWS(HD_, TO_, true); else KV_ROWS(HD_, TO_, false); } while (0)
    if (hd == 128) { if (to_cache) KV_ROWS2(128, true); else KV_ROWS2(128, false); }
    else           { if (to_cache) KV_ROWS2(64, true);  else KV_ROWS2(64, false); }
#undef KV_ROWS2
#undef KV_ROWS
}

// ------------------------------------------------------------------------------------------
// Small copies out of the padded internal buffers into the caller's dense outputs.
__global__ void k_copy_row_stats(const float4* __restrict__ src, float4* __restrict__ dst, int B, int T, int Tp) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < B * T) dst[i] = src[(i / T) * Tp + i % T];
}
void launch_copy_row_stats(const float4* src, float4* dst, int B, int T, int Tp, hipStream_t s) {
    hipLaunchKernelGGL(k_copy_row_stats, dim3((B * T + 255) / 256), dim3(256), 0, s, src, dst, B, T, Tp);
}

__global__ void k_fill_i32(int32_t* p, int32_t v, int n) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}
void launch_fill_i32(int32_t* p, int32_t v, int n, hipStream_t s) {
    hipLaunchKernelGGL(k_fill_i32, dim3((n + 255) / 256), dim3(256), 0, s, p, v, n);
}

// two arrays in one launch (a sequence's root token and its candidates: bound by the launch)
__global__ void k_copy_i32(const int32_t* __restrict__ src, int32_t* __restrict__ dst, int n, const int32_t* __restrict__ src2,
                           int32_t* __restrict__ dst2, int n2) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) dst[i] = src[i];
    if (i < n2) dst2[i] = src2[i];
}
void launch_copy_i32(const int32_t* src, int32_t* dst, int n, const int32_t* src2, int32_t* dst2, int n2, hipStream_t s) {
    const int most = n > n2 ? n : n2;
    hipLaunchKernelGGL(k_copy_i32, dim3((most + 255) / 256), dim3(256), 0, s, src, dst, n, src2, dst2, n2);
}
// dst[0 .. n) = the values, which travel with the launch: nothing of the caller's is read later
__global__ void k_set_i32(SeqList v, int32_t* __restrict__ dst, int n) {
    if (threadIdx.x < n) dst[threadIdx.x] = v.seq[threadIdx.x];
}
void launch_set_i32(const int32_t* v, int32_t* dst, int n, hipStream_t s) {
    SeqList l = {};
    for (int i = 0; i < n; ++i) l.seq[i] = v[i];
    hipLaunchKernelGGL(k_set_i32, dim3(1), dim3(SD_MAX_BATCH), 0, s, l, dst, n);
}

// Prompt chunks commit every row: slots are the identity, the count is the chunk length. (src_slots, n_accept and n_old
// by sequence of the pass, kv_len by sequence of the cache.)
__global__ void k_prefill_commit_setup(ChainArgs ca, RowMap rm, int B, int Tp, int32_t* __restrict__ src_slots,
                                       int32_t* __restrict__ n_accept, int32_t* __restrict__ n_old,
                                       int32_t* __restrict__ kv_len, int32_t* __restrict__ fin_rows, int n_fin, SeqList last) {
    const int b = blockIdx.x, j = threadIdx.x;
    if (b == 0 && j < n_fin) fin_rows[j] = last.seq[j];
    if (j < Tp) src_slots[(size_t)b * Tp + j] = j;
    if (j == 0) {
        const int sq = rm.seq[b], n = kv_len[sq];
        n_old[b] = n;
        n_accept[b] = ca.len[b];
        kv_len[sq] = n + ca.len[b];
    }
}
void launch_prefill_commit_setup(const ChainArgs& ca, const RowMap& rm, int B, int Tp, int32_t* src_slots, int32_t* n_accept,
                                 int32_t* n_old, int32_t* kv_len, int32_t* fin_rows, int n_fin, const SeqList& last, hipStream_t s) {
    hipLaunchKernelGGL(k_prefill_commit_setup, dim3(B), dim3(SD_MAX_TREE), 0, s, ca, rm, B, Tp, src_slots, n_accept, n_old,
                       kv_len, fin_rows, n_fin, last);
}

// commit stage alone: the count of every sequence clamped to [0, width] (0 where bit b of `held` is not set: the last pass
// left no rows of it), old length noted, new length set
__global__ void k_commit_setup(const int32_t* __restrict__ n_rows, int width, uint32_t held, int B, int32_t* __restrict__ n_accept,
                               int32_t* __restrict__ n_old, int32_t* __restrict__ kv_len) {
    const int b = threadIdx.x;
    if (b >= B) return;
    const int a = (held >> b) & 1u ? min(max(n_rows[b], 0), width) : 0, n = kv_len[b];
    n_accept[b] = a;
    n_old[b] = n;
    kv_len[b] = n + a;
}
void launch_commit_setup(const int32_t* n_rows, int width, uint32_t held, int B, int32_t* n_accept, int32_t* n_old,
                         int32_t* kv_len, hipStream_t s) {
    hipLaunchKernelGGL(k_commit_setup, dim3(1), dim3(SD_MAX_BATCH), 0, s, n_rows, width, held, B, n_accept, n_old, kv_len);
}

// root_tok of the sequences whose prompt just ended: arg-max of their last rows' logits
__global__ void k_pick_root(const float2* __restrict__ best, int nch, int32_t* __restrict__ root_tok, int n, SeqList sl) {
    const int i = threadIdx.x;
    if (i < n) root_tok[sl.seq[i]] = best_of_chunks(best + (size_t)i * nch, nch);
}
void launch_pick_root(const float2* best, int V, int32_t* root_tok, int n, const SeqList& sl, hipStream_t s) {
    hipLaunchKernelGGL(k_pick_root, dim3(1), dim3(SD_MAX_BATCH), 0, s, best, rank_chunks(V), root_tok, n, sl);
}
