// How the projections are cut into workgroups: plain host arithmetic on sizes, no HIP in here.
#pragma once
#include <stdint.h>
#include <string.h>

#define SK_MAX_WG 256       // one workgroup of 8 waves per CU (at 94 registers k_gemm_sk leaves room for two: not tried as a plan)

// How one GEMM shape is launched (made once per shape at model creation).
struct GemmPlan {
    int MB, KB, NB;
    int G, NG;               // workgroups, 256-column groups
    int upw, rem;            // units per workgroup; the first `rem` workgroups take one more
    int slots;               // slots the output buffer must hold
    int uniform;             // 1: every column group has exactly `slots` contributors
    int CG, S;               // four / eight row blocks as launched by launch_gemm: column groups of CG blocks, each
                             // split into S segments of the contraction (workgroup = group * S + segment, slot =
                             // segment); 0 for one and two row blocks. The fields above then describe the balanced
                             // split that the persistent layer kernel walks at eight row blocks.
    int RT, MT;              // prompt passes of more than 256 rows: RT tiles of MT row blocks each (MB = all of them), one
                             // workgroup per tile, column group and segment; 0 otherwise
    int chain;               // ... whose sums of products are folded away every `chain` contraction blocks (0: they are not)
    int slots_max;           // slots the output buffer must hold for either
    int32_t* cnt_dev;        // [NG] contributors per column group (device)
    int32_t* slot0_dev;      // [G] slot of every workgroup's first segment (device)
};

// Four and eight row blocks (k_gemm_rows): the width of a column group, CG blocks, and the number of segments S the
// contraction is split into, S a divisor of KB, at most 16. Cost of a candidate in shader cycles, from the kernel's
// measured pace: a step costs its MFMAs (two waves per SIMD, 2 x CPW MFMAs of 32 cycles each) plus about 300 cycles
// of hand-over; a workgroup runs KB / S steps (rounded up to the ring), the grid ceil(groups x S / 256) rounds; the S
// partial tiles are written at the end of the kernel and read by the consumer at about 2500 bytes per cycle each
// way. Narrow groups buy workgroups and few slots for the matrices with few columns (O and down projection at the
// 7B shape, 256 rows: 4 blocks x 8 segments instead of 8 x 16: 22 us against 26, 41 against 43, and the consumer
// reads half as much); six-block groups fill the chip where eight-block ones leave a quarter of it idle (QKV: 64
// groups x 4 = 256 workgroups, 45 us against 55 with 48 x 4; gate/up 115 x 2 = 230 against 86 x 2 = 172: 76 against 89).
static inline double gemm_plan_rows(GemmPlan* p) {      // -> the cost
    const int MT = p->MB;
    static const int widths8[] = {8, 6, 4}, widths4[] = {8, 4};
    const int* widths = MT == 8 ? widths8 : widths4;
    const int n_widths = MT == 8 ? 3 : 2;
    double best = 0;
    for (int wi = 0; wi < n_widths; ++wi) {
        const int CG = widths[wi], groups = (p->NB + CG - 1) / CG;
        for (int S = 1; S <= 16 && S <= p->KB; ++S) {
            if (p->KB % S) continue;
            const int G = groups * S, rounds = (G + SK_MAX_WG - 1) / SK_MAX_WG;
            const int steps = (p->KB / S + 3) / 4 * 4;
            const double step_cycles = 16.0 * CG * MT + 300.0;
            const double tile_bytes = (double)S * MT * 32 * p->NB * 32 * 4;
            const double cost = rounds * steps * step_cycles + 2.0 * tile_bytes / 2500.0;
            if (p->CG == 0 || cost < best) { best = cost; p->CG = CG; p->S = S; }
        }
    }
    if (p->S > p->slots_max) p->slots_max = p->S;
    return best;
}

// Prompt passes of more than 256 rows: tiles of eight or four row blocks, the cost of gemm_plan_rows over all of them, and
// 6000 cycles (launch, first loads, stores) per round of workgroups. With this many rows a projection needs fewer segments to
// fill the chip (7B shape, 1024 rows: QKV and gate/up one, O and down two, where 256 rows have two to eight), so fewer partial
// tiles are written and read; the weights are read once per pass.
// 7B shape, a prompt of 1500 tokens through four layers: 6560 us in six passes of up to 256 rows, 5620 in passes of 1024 and
// 476 (5430 with chains of any length). The launches themselves run at what the card's power allows for dense data, 0.97-1.05 PFLOP/s of two-term work at
// 256 and at 1024 rows alike (1.26-1.36 with operands of zeros): what is saved lies between them.
//
// Fewer segments are longer sums, and a sum that is rounded at every contraction block strays with its length: with one
// segment for 256 blocks the QKV sums were 4.5 % further from 64 bits than with the four of a 256-row pass. So no chain of
// products is longer than in a 256-row pass of the same matrix: a workgroup adds its sums to a second set ("folds") that often.
// The tiles with room for a second set can (registers, and LDS for the tile of eight row blocks and six columns); the tile
// of eight by eight has none and is taken only with segments that are short enough as they are (7B shape, 1024 rows: the down
// projection in eight by eight, four segments of 172 blocks, 170 us; in eight by four, two segments of five chains, 193).
static inline bool gemm_tile_folds(int MT, int CG) { return CG * MT <= 32 || (MT == 8 && CG == 6); }
// Longest chain of a 256-row pass, in contraction blocks.
static inline int gemm_chain_limit(int KB, int NB) {
    GemmPlan q;
    memset(&q, 0, sizeof(q));
    q.MB = 8; q.KB = KB; q.NB = NB;
    gemm_plan_rows(&q);
    return KB / q.S;
}
static inline void gemm_plan_prompt(GemmPlan* p, int MB, int KB, int NB, double* cycles) {
    memset(p, 0, sizeof(*p));
    p->MB = MB; p->KB = KB; p->NB = NB;
    static const int widths8[] = {8, 6, 4}, widths4[] = {8, 4};
    const int limit = gemm_chain_limit(KB, NB);
    double best = 0;
    for (int MT = 8; MT >= 4; MT /= 2)
        for (int wi = 0; wi < (MT == 8 ? 3 : 2); ++wi) {
            const int CG = MT == 8 ? widths8[wi] : widths4[wi], groups = (NB + CG - 1) / CG, RT = (MB + MT - 1) / MT;
            for (int S = 1; S <= 4 && S <= KB; ++S) {
                if (KB % S) continue;
                const int n = KB / S;
                int chain = 0;
                if (n > limit) {                       // even chains, in the kernels' grain of eight blocks
                    if (!gemm_tile_folds(MT, CG)) continue;
                    const int most = limit < 8 ? 8 : limit / 8 * 8, chains = (n + most - 1) / most;
                    if (chains > 1) chain = ((n + chains - 1) / chains + 7) / 8 * 8;
                }
                const int rounds = ((groups * S + 7) / 8 * RT + 31) / 32, steps = (n + 3) / 4 * 4;      // (an XCD's)
                const double tile_bytes = (double)S * MB * 32 * NB * 32 * 4;
                const double folds = chain ? (n - 1) / chain * 50.0 * CG * MT : 0.0;
                const double cost = rounds * (steps * (16.0 * CG * MT + 300.0) + folds + 6000.0) + 2.0 * tile_bytes / 2500.0;
                if (p->CG == 0 || cost < best) { best = cost; p->CG = CG; p->S = S; p->MT = MT; p->RT = RT; p->chain = chain; }
            }
        }
    p->slots = p->slots_max = p->S;
    p->uniform = 1;
    *cycles = best;
}
