// Plain host arithmetic on sizes: no HIP in here.
#pragma once

// How the attention of a pass is cut into workgroups (one resident per compute unit: the kernel
// takes the whole LDS). A group is one (sequence, head, query-block group); it gets `ncparts` cache
// parts of `per` 32-row blocks each, sized from the host's bound on the sequence lengths, and the
// tree blocks go to a part of their own while the chip has room for it (short contexts) or to the
// last cache part (long contexts).
// tree_sep: parts that hold tree blocks only: 0 (the last cache part takes them), 1, or, when the attention launch
// builds the tree's keys and values itself (one query group of two blocks: split_ok), one per tree block, so that the
// building is shared by two workgroups.
struct AttnGeom { int ncparts, per, tree_sep, nparts; };
static inline AttnGeom attn_geometry(int n_heads, int max_parts, int B, int Tp, int n_hi, bool split_ok, bool ragged) {
    auto ceil_div = [](int a, int b) { return (a + b - 1) / b; };
    const int nblk = ceil_div(n_hi, 32);
    const int TB = Tp / 32, TG = (TB % 2 == 0) ? TB / 2 : TB;
    const int groups = B * n_heads * TG;
    int P = 256 / groups;                                  // parts per group that fit the chip at once
    if (P < 1) P = 1;
    if (P > max_parts) P = max_parts;
    AttnGeom g;
    if (nblk == 0) { g.ncparts = 0; g.per = 1; g.tree_sep = 1; g.nparts = 1; return g; }
    // A batch with one workgroup per (sequence, head) lasts as long as its longest sequence: when the lengths are ragged,
    // two parts that share every sequence's own blocks evenly (per = 0). Launch at eight 7B-shaped sequences of 1024 - 4096
    // rows: plain decoding 88 -> 78 us, 32-node trees 88 -> 82; one of 4096 beside seven of 32 rows 56 -> 36; but eight of
    // 2560 rows 74.6 -> 77.6, so not where they are alike. (Three and four parts 85 and 95 us: one workgroup of this
    // kernel fits a compute unit, and held to 256 registers, so that two fit, it spills: 107 us.)
    if (P == 1 && TB == 1 && ragged && nblk >= 8) {
        g.tree_sep = 0;
        g.ncparts = g.nparts = 2;
        g.per = 0;
        return g;
    }
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
// rules that rest on the attention launch building the tree's keys itself apply there: no second tree part, no even parts.
static inline AttnGeom attn_geometry_of_pass(bool fused, int n_heads, int max_parts, int B, int Tp, int n_hi, bool ragged) {
    return attn_geometry(n_heads, max_parts, B, Tp, n_hi, !fused && Tp == 64, !fused && ragged);
}
