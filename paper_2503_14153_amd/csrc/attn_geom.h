// Plain host arithmetic on sizes: no HIP in here.
#pragma once
#include <stdint.h>

// How the attention of a pass is cut into workgroups (one resident per compute unit where a group has two query blocks: such a
// one takes the whole LDS; with one block two fit, which attn_split uses). A group is one (sequence, head, query-block group); it gets `ncparts` cache
// parts of `per` 32-row blocks each, sized from the host's bound on the sequence lengths, and the
// tree blocks go to a part of their own while the chip has room for it (short contexts) or to the
// last cache part (long contexts).
// tree_sep: parts that hold tree blocks only: 0 (the last cache part takes them), 1, or, when the attention launch
// builds the tree's keys and values itself (one query group of two blocks: split_ok), one per tree block, so that the
// building is shared by two workgroups.
struct AttnGeom { int ncparts, per, tree_sep, nparts; };
static inline AttnGeom attn_geometry(int n_heads, int max_parts, int B, int Tp, int n_hi, bool split_ok) {
    auto ceil_div = [](int a, int b) { return (a + b - 1) / b; };
    const int nblk = ceil_div(n_hi, 32);
    const int TB = Tp / 32, TG = (TB % 2 == 0) ? TB / 2 : TB;
    const int groups = B * n_heads * TG;
    int P = 256 / groups;                                  // parts per group that fit the chip at once
    if (P < 1) P = 1;
    if (P > max_parts) P = max_parts;
    AttnGeom g;
    if (nblk == 0) { g.ncparts = 0; g.per = 1; g.tree_sep = 1; g.nparts = 1; return g; }
    const int by_work = ceil_div(nblk, 4);                 // at least one block per wave
    const int ntp = (split_ok && TB == 2 && P >= 3) ? 2 : 1;
    // The tree keeps parts of its own while the cache parts are short: up to eight blocks per cache part, or, when a
    // single sequence has the chip (eight parts per head, of which the tree's one or two idle while the others stream),
    // up to forty: there the launch without the rotary stage before it wins up to ~8 k rows (64-node tree, step at
    // 1.5 / 3 / 6 k rows: 5.18 -> 5.06, 5.25 -> 5.20, 5.55 -> 5.47 ms; at 16 k rows 6.40 -> 6.45, so not there).
    const int short_mult = P >= 8 ? 40 : 8;
    if (P >= 2 && nblk <= short_mult * (P - ntp)) {        // short: the tree beside the cache parts
        // (two blocks per wave before another part is opened: every part repeats the queries' set-up and adds a term
        // to the merge; 7B shape, 64-node tree over 512-1800 rows: attention launch 18.4 -> 16.8 us, step -1 %)
        const int by_two = ceil_div(nblk, 8);
        g.tree_sep = ntp;
        g.ncparts = P - ntp < by_two ? P - ntp : by_two;
    } else {
        g.tree_sep = 0;
        g.ncparts = P < by_work ? P : by_work;
    }
    g.per = ceil_div(nblk, g.ncparts);
    g.ncparts = ceil_div(nblk, g.per);
    g.nparts = g.ncparts + g.tree_sep;
    return g;
}

// The geometry of a pass. The persistent layer kernel (fused) keeps the rotary stage as a phase of its own, so none of the
// rules that rest on the attention launch building the tree's keys itself apply there: no second tree part, no parts per
// sequence. ragged: a batch whose sequences are to be cut one by one, if they have one query block each: per = 0 says that
// attn_split tells how (two parts, or more or fewer).
static inline AttnGeom attn_geometry_of_pass(bool fused, int n_heads, int max_parts, int B, int Tp, int n_hi, bool ragged) {
    if (ragged && !fused && Tp == 32) return AttnGeom{2, 0, 0, 2};
    return attn_geometry(n_heads, max_parts, B, Tp, n_hi, !fused && Tp == 64);
}

// Batches of one query block per sequence (trees of up to 32 nodes, plain decoding): every sequence gets parts in proportion
// to its length, and shares its own blocks, as many as the device says it has, evenly among them. One entry per (sequence, part),
// each a workgroup per head; n = 0: not used.
#define ATTN_SPLIT_MAX 64
struct AttnSplit {
    uint32_t slot[ATTN_SPLIT_MAX];       // sequence | part << 8 | parts of the sequence << 16
    int n, max_parts;                    // entries; parts of the sequence that has the most
};
// The smallest block count per part, q >= 8 (two a wave), with which the parts of all sequences number `want` at most.
static inline int attn_parts(int len, int q) {
    const int parts = ((len + 31) / 32 + q - 1) / q;
    return parts < 1 ? 1 : parts > 15 ? 15 : parts;
}
static inline int attn_split_q(int B, const int* len, int want) {
    for (int q = 8;; ++q) {
        int total = 0;
        for (int b = 0; b < B; ++b) total += attn_parts(len[b], q);
        if (total <= want || q >= 1 << 20) return q;
    }
}
// len: the host's bounds. One workgroup per compute unit, or two (both fit; no more: a second round costs more than any
// balance gains), whichever the measured pace says is sooner done: a launch takes 9.4 us, 2.5 more with two per unit, and the
// longer of its bytes (2.73 ns a block) and the blocks of its longest workgroup (0.5 us each alone on a unit, 0.8 beside
// another). 7B shape, plain decoding, one / two per unit, us: eight sequences of 2656 rows 67.4 / 69.9; of 1024 32.1 / 35.9;
// of 1024 - 4096 80 / 75 (79 with two even parts each, as it was); five of 150 - 2100 25.4 / 27.8 (32); three per unit 84.
static inline AttnSplit attn_split(int n_heads, int B, const int* len) {
    AttnSplit s = {};
    double best = 0;
    int best_q = 1;
    for (int k = 1; k <= 2; ++k) {
        int want = 256 * k / n_heads;
        if (want > ATTN_SPLIT_MAX) want = ATTN_SPLIT_MAX;
        if (want < B) want = B;
        const int q = attn_split_q(B, len, want);
        int longest = 0, blocks = 0;
        for (int b = 0; b < B; ++b) {
            const int nb = (len[b] + 31) / 32, parts = attn_parts(len[b], q), each = (nb + parts - 1) / parts;
            blocks += nb;
            if (each > longest) longest = each;
        }
        const double stream = blocks * n_heads * 2.73, chain = longest * (k == 1 ? 500.0 : 800.0);
        const double cost = 9400.0 + 2500.0 * (k - 1) + (stream > chain ? stream : chain);
        if (k == 1 || cost < best) { best = cost; best_q = q; }
    }
    for (int b = 0; b < B; ++b) {
        const int parts = attn_parts(len[b], best_q);
        if (parts > s.max_parts) s.max_parts = parts;
        for (int p = 0; p < parts; ++p) s.slot[s.n++] = (uint32_t)b | (uint32_t)p << 8 | (uint32_t)parts << 16;
    }
    return s;
}

// One workgroup per (sequence, head, row block) instead of parts (attn_whole.hip, which has the figures behind this line): two
// row blocks or more, at least 64 such workgroups, and no more blocks per workgroup than 18 where there are 64 of them, 36 where
// there are 128, and up to 72. One fits a compute unit: beyond 256 of them a second round halves that (13B shape, two 128-node
// trees, 320 workgroups: 36 blocks level, 67 blocks 2.3 % of the step slower), and with two row blocks per sequence, where the
// parts' launch makes its queries and tree keys itself in one round, it never pays (four 64-node trees over 100 / 1000 / 2500
// rows 0.6 / 2.9 / 5.8 % slower).
// Tp counts what a prompt's layout has room for, not the rows that exist. Counted by those, the last 9 to 32 rows of a prompt
// would go to the parts' launch, and they are 4-7 % faster here over up to 1000 rows (7B and 13B shape; 33 to 100 rows level).
static inline bool attn_whole_pays(int n_heads, int B, int Tp, int n_hi) {
    const int groups = B * n_heads * (Tp / 32), rounds = (groups + 255) / 256, blocks = (n_hi + 31) / 32 + Tp / 32;
    if (Tp < 64 || groups < 64 || (rounds > 1 && Tp == 64)) return false;
    return blocks * rounds * 64 <= 18 * (groups < 256 ? groups : 256);
}
// Parts of a (sequence, head, row block) in attn_whole.hip: 1 where one workgroup takes all of it (above), 0 where attn.hip's
// parts are faster, or, for sequences of two row blocks each, as many as fill the chip with workgroups of one row block:
// three or four, of up to 33 blocks. Two query blocks share a wave in attn.hip, which halves its reads of a long cache; over a
// short one its four waves have a block or two each, one after the other, and these have eight. Steps of four layers, 7B shape, 64
// nodes, us, attn.hip / here: 700 rows 702 / 694 (32 layers: 4652 / 4645), 1100 696.5 / 688, 2200 712 / 701, 3000 729 / 725, 4200 732 / 725, 6000 761 / 763,
// 16384 873 / 895; 13B shape, two layers: 1200 rows 537 / 524, 2000 541 / 533, 4096 561 / 569. Two sequences of 16 to 20 heads and three
// of 11 to 13 over 700 to 4000 rows, ragged ones too: up to 4 % of the step faster; four of 8 to 10 heads of 64 dims 0 to 6 % faster, of 128 dims
// from 2 % faster (700 rows) to 2 % slower (nine heads, 2900 rows). Two parts are level.
// All parts and row blocks of a (sequence, head) run on one XCD and those are dealt to the eight in turn, so the chip is full when
// the XCD with the most of them is: 41 and 42 (sequence, head) pairs, six on two of the XCDs, are 36 workgroups for 32 compute units
// there (one sequence of 42 heads over 700 / 2000 / 2900 rows 890 / 913 / 924 in attn.hip, 903 / 941 / 961 here; two of 21 heads, three of 14 the same).
static inline int attn_whole_parts(int n_heads, int B, int Tp, int n_hi) {
    if (attn_whole_pays(n_heads, B, Tp, n_hi)) return 1;
    const int pairs = B * n_heads, blocks = (n_hi + 31) / 32 + Tp / 32;
    if (Tp != 64 || pairs < 32) return 0;
    const int P = 32 / ((pairs + 7) / 8 * 2);          // 32 compute units of an XCD
    return P >= 3 && blocks <= 33 * P ? P : 0;
}
// The same for joined prompt passes, whose workgroups come in several rounds: chunks of Tp rows over at most n_hi others. No more
// than 32 blocks, which is 1024 rows of one prompt. Two layers, us, attn.hip and merge / here: 7B shape, 512 tokens 894 / 882, 800
// 1645 / 1609, 1024 1697 / 1689, four prompts of 100 - 375 1673 / 1642; 13B shape, 400 tokens 1324 / 1294, 1024 2616 / 2593; beyond, 2048
// tokens of the 7B shape 3348 / 3388, 4096 6831 / 7263. Few heads ask for no line of their own: 4, 8 and 16 heads, prompts of 300 to 1000 tokens
// and batches of two to eight in chunks of 32 to 256 rows take 0.92 to 0.99 of the time; eight prompts of 33 tokens, chunks of 32 rows, 0.96 to 1.005.
static inline bool attn_whole_pays_prompt(int Tp, int n_hi) { return (n_hi + 31) / 32 + Tp / 32 <= 32; }
