// How the projections are cut into workgroups: plain host arithmetic on sizes, no HIP in here.
#pragma once
#include <stdint.h>
#include <string.h>

#include <vector>

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

// Four and eight row blocks (k_gemm_tile): the width of a column group, CG blocks, and the number of segments S the
// contraction is split into, S a divisor of KB, at most 16. Cost of a candidate in shader cycles: a step costs its MFMAs
// (CG x MT / 2 of 32 cycles each per SIMD) plus 300 cycles of everything else, the pace of the kernel before this one, which
// needs 177 at eight by six and 233 at four by eight; a workgroup runs KB / S steps (rounded up to four), the grid
// ceil(groups x S / 256) rounds; the S
// partial tiles are written at the end of the kernel and read by the consumer at about 2500 bytes per cycle each
// way. Narrow groups buy workgroups and few slots for the matrices with few columns (O and down projection at the
// 7B shape, 256 rows: 4 blocks x 8 segments instead of 8 x 16: 22 us against 27, 43 against 45, and the consumer
// reads half as much); six-block groups fill the chip where eight-block ones leave a quarter of it idle (QKV: 64
// groups x 4 = 256 workgroups, 48 us against 54 with 48 x 4; gate/up 115 x 2 = 230 against 86 x 2 = 172: 83 against 94).
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
// 7B shape, a prompt of 1500 tokens through four layers: 6130 us in six passes of up to 256 rows, 5076 in passes of 1024 and
// 476 (4708 with chains of any length, see below).
//
// Fewer segments are longer sums, and a sum that is rounded at every contraction block strays with its length: with one
// segment for 256 blocks the QKV sums were 4.5 % further from 64 bits than with the four of a 256-row pass. So no chain of
// products is longer than in a 256-row pass of the same matrix: a workgroup adds its sums to a second set ("folds") that often.
// The tile of eight by eight blocks has room for half of a second set and puts the rest into its output: dear, but with few
// folds the tile that moves the fewest bytes per product is still the fastest (7B shape, 1024 rows, down projection: eight by
// four, two segments of five chains each 200 us; eight by eight, four segments of three chains 180).
// Longest chain of a 256-row pass, in contraction blocks.
static inline int gemm_chain_limit(int KB, int NB) {
    GemmPlan q;
    memset(&q, 0, sizeof(q));
    q.MB = 8; q.KB = KB; q.NB = NB;
    gemm_plan_rows(&q);
    return KB / q.S;
}
// gate_up: the matrix is the gate/up projection (gemm_plan_swiglu below: half the bytes written, none read again).
static inline void gemm_plan_prompt(GemmPlan* p, int MB, int KB, int NB, double* cycles, bool gate_up = false) {
    memset(p, 0, sizeof(*p));
    p->MB = MB; p->KB = KB; p->NB = NB;
    static const int widths8[] = {8, 6, 4}, widths4[] = {8, 4};
    const int limit = gemm_chain_limit(KB, NB);
    const int most = limit < 8 ? 8 : limit / 8 * 8;        // even chains, in the kernels' grain of eight blocks
    auto even = [&](int n) { const int chains = (n + most - 1) / most; return chains > 1 ? ((n + chains - 1) / chains + 7) / 8 * 8 : 0; };
    double best = 0;
    for (int MT = 8; MT >= 4; MT /= 2)
        for (int wi = 0; wi < (MT == 8 ? 3 : 2); ++wi) {
            const int CG = MT == 8 ? widths8[wi] : widths4[wi], groups = (NB + CG - 1) / CG, RT = (MB + MT - 1) / MT;
            for (int S = 1; S <= 4 && S <= KB; ++S) {
                if (KB % S) continue;
                const int n = KB / S;
                const int chain = n > limit ? even(n) : 0;
                const int rounds = ((groups * S + 7) / 8 * RT + 31) / 32, steps = (n + 3) / 4 * 4;      // (an XCD's)
                const double tile_bytes = (double)S * MB * 32 * NB * 32 * 4 * (gate_up && MT == 8 && CG == 6 && S == 1 ? 0.25 : 1.0);
                const double folds = chain ? (n - 1) / chain * (MT * CG == 64 ? 160.0 : 50.0) * CG * MT : 0.0;
                const double cost = rounds * (steps * (16.0 * CG * MT + 300.0) + folds + 6000.0) + 2.0 * tile_bytes / 2500.0;
                if (p->CG == 0 || cost < best) { best = cost; p->CG = CG; p->S = S; p->MT = MT; p->RT = RT; p->chain = chain; }
            }
        }
    p->slots = p->slots_max = p->S;
    p->uniform = 1;
    *cycles = best;
}
// The gate/up projection of a prompt pass whose workgroups see whole sums of 96 gate columns and the up columns that belong to
// them: it writes silu(gate) * up, as the next projection's operand, instead of the sums (k_gemm_tile).
static inline bool gemm_plan_swiglu(const GemmPlan& p) { return p.RT && p.MT == 8 && p.CG == 6 && p.S == 1; }

// Time of a layer of a prompt pass, us, from its rows and its four projections (sh: contraction and column blocks of each). Up to
// 64 rows the weights' bytes; up to 256 the cost above at 1950 cycles per us, with 60000 cycles for the layer's other launches;
// joined passes at 1700 (less of what they lose is in the model). Measured, us a layer, 7B / 13B shape (in brackets what this says):
// 8 rows 90 / 145 (103 / 153), 32 rows 106 / 152, 64 rows 132 / 171 (132 / 176), 128 rows 164 / 221 (178 / 222), 256 rows 237 / 336
// (253 / 352); joined 288 rows 384 / 510 (443 / 623), 320 387 / 517 (447 / 631), 512 407 / 631 (470 / 711), 640 614 / 883 (705 / 983), 768
// 707 / 905 (790 / 995), 1024 812 / 1253 (834 / 1291). It was fitted to the kernel before: the times are up to a fifth too
// long, most for the shorter joined passes, so that some prompts are cut where one pass would be sooner done (13B shape, 512
// tokens: two passes of 256 rows 672, one 631). A remainder of a few rows is right to run alone (257 tokens: 257 rows as one pass
// take about 384 / 510, 256 rows and one 330 / 480).
static inline double prompt_pass_us(const int (*sh)[2], int rows) {
    double bytes = 0, cycles = 60000;
    const int mb = (rows + 31) / 32;
    for (int i = 0; i < 4; ++i) {
        bytes += (double)sh[i][0] * sh[i][1] * 1024;
        GemmPlan p;
        double c = 0;
        if (mb > 8) {
            gemm_plan_prompt(&p, mb, sh[i][0], sh[i][1], &c, i == 2);
        } else {
            memset(&p, 0, sizeof(p));
            p.MB = mb > 4 ? 8 : 4; p.KB = sh[i][0]; p.NB = sh[i][1];
            c = gemm_plan_rows(&p);
        }
        cycles += c;
    }
    return mb <= 1 ? bytes / 4.6e6 + 15 : mb == 2 ? bytes / 5.2e6 + 54 : mb <= 8 ? cycles / 1950 : cycles / 1700;
}

// Which of n passes run as one: the partition into runs of neighbours with the smallest sum of times. rows(i, k): the rows of
// passes [i, i + k) as one, 0 where they cannot be (and where no longer run can); us(rows): the time. -> the runs' lengths.
template <class Rows, class Us>
static inline std::vector<int> prompt_runs(int n, Rows&& rows, Us&& us) {
    std::vector<double> best(n + 1, 0.0);               // of the passes from i on
    std::vector<int> take(n, 1), runs;
    for (int i = n - 1; i >= 0; --i)
        for (int k = 1; i + k <= n; ++k) {
            const int r = rows(i, k);
            if (r == 0) break;
            const double t = us(r) + best[i + k];
            if (k == 1 || t < best[i]) { best[i] = t; take[i] = k; }
        }
    for (int i = 0; i < n; i += take[i]) runs.push_back(take[i]);
    return runs;
}
