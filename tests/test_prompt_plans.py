"""How the projections of prompt passes are cut (gemm_plan.h), on the CPU: no chain of products is longer than a 256-row pass's of
the same matrix, and the chains are what the kernels can walk."""
import ctypes as C
import os
import random
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CODE = """
#include "gemm_plan.h"
extern "C" int limit(int KB, int NB) { return gemm_chain_limit(KB, NB); }
extern "C" void plan(int MB, int KB, int NB, int gate_up, int* out) {
    GemmPlan p;
    double cycles;
    gemm_plan_prompt(&p, MB, KB, NB, &cycles, gate_up);
    const int f[] = {p.MT, p.CG, p.S, p.RT, p.chain, p.slots_max};
    for (int i = 0; i < 6; ++i) out[i] = f[i];
}
extern "C" double us(const int* sh, int rows) { return prompt_pass_us((const int(*)[2])sh, rows); }
extern "C" int runs(const int* sh, int n, const int* rows, int* out) {     // one sequence: passes of 256 rows, then what is left
    const auto total = [&](int i, int k) {
        int M = 0;
        for (int j = i; j < i + k; ++j) M += rows[j];
        return k > 1 && M > 1024 ? 0 : M;
    };
    const std::vector<int> r = prompt_runs(n, total, [&](int m) { return prompt_pass_us((const int(*)[2])sh, m); });
    for (size_t i = 0; i < r.size(); ++i) out[i] = r[i];
    return (int)r.size();
}
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("plans")
    (d / "plans.cpp").write_text(CODE)
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_2503_14153_amd", "csrc"), str(d / "plans.cpp"), "-o", str(d / "plans.so")],
                   check=True)
    return C.CDLL(str(d / "plans.so"))


def plan(lib, MB, KB, NB, gate_up=False):
    out = (C.c_int * 6)()
    lib.plan(MB, KB, NB, gate_up, out)
    return dict(zip(["MT", "CG", "S", "RT", "chain", "slots"], out))


def shapes():
    """(d_model, d_ffn) -> the four projections in blocks of 16 inputs and 32 outputs, and whether it is gate/up."""
    rng = random.Random(5)
    for d, F in [(4096, 11008), (5120, 13824), (256, 688), (64, 16)] + [(32 * rng.randint(1, 256), 16 * rng.randint(1, 1800)) for _ in range(60)]:
        gu = 2 * (-(-F // 32))
        yield from [(d // 16, 3 * d // 32, 0), (d // 16, d // 32, 0), (d // 16, gu, 1), (F // 16, d // 32, 0)]


def test_chains_are_no_longer_than_in_a_256_row_pass(lib):
    """As launched: S segments of n contraction blocks, S partial tiles, the sums folded away every `chain` blocks."""
    folds = {}
    for KB, NB, gate_up in shapes():
        limit = lib.limit(KB, NB)
        for MB in range(9, 33):
            p = plan(lib, MB, KB, NB, gate_up)
            n, chain = KB // p["S"], p["chain"]
            assert KB % p["S"] == 0 and p["S"] <= 4 and p["slots"] == p["S"] and p["MT"] * p["RT"] >= MB
            assert min(n, chain or n) <= max(limit, 8), (KB, NB, MB, p, limit)
            if chain:
                tile = (p["MT"], p["CG"])
                folds[tile] = folds.get(tile, 0) + 1
                assert chain % 8 == 0 and chain < n            # (the kernels' grain; there is something to fold)
    assert sum(folds.values()) > 100 and folds[8, 8] > 20 and folds[8, 6] > 20, folds


def test_the_plan_of_a_tile_that_folds_says_what_is_launched(lib):
    """1024 rows of the 7B shape, down projection: tiles of eight by eight blocks, four segments of 172 contraction blocks, each
    in chains of 64, 64 and 44 (a 256-row pass has chains of 86)."""
    p = plan(lib, 32, 688, 128)
    assert lib.limit(688, 128) == 86
    assert p == {"MT": 8, "CG": 8, "S": 4, "RT": 4, "chain": 64, "slots": 4}


def projections(d, F):
    return [d // 16, 3 * d // 32, d // 16, d // 32, d // 16, 2 * -(-F // 32), -(-F // 16), d // 32]


def cut(lib, d, F, tokens):
    """Rows of the passes that a prompt of so many tokens becomes."""
    rows = [256] * (tokens // 256) + [tokens % 256] * (tokens % 256 > 0)
    out = (C.c_int * len(rows))()
    n = lib.runs((C.c_int * 8)(*projections(d, F)), len(rows), (C.c_int * len(rows))(*rows), out)
    ends = [sum(out[:i]) for i in range(n + 1)]
    assert ends[-1] == len(rows)
    return [sum(rows[a:b]) for a, b in zip(ends, ends[1:])]


# a pass of its own costs a short remainder its weights; joined, it costs all rows a coarser tile (both sides measured: gemm_plan.h)
@pytest.mark.parametrize("d,F,tokens,passes", [
    (4096, 11008, 257, [256, 1]), (4096, 11008, 300, [256, 44]), (4096, 11008, 320, [256, 64]), (4096, 11008, 512, [512]),
    (4096, 11008, 640, [512, 128]), (4096, 11008, 1024, [1024]), (4096, 11008, 1500, [1024, 476]),
    (5120, 13824, 257, [256, 1]), (5120, 13824, 300, [256, 44]), (5120, 13824, 512, [256, 256]), (5120, 13824, 560, [256, 256, 48]),
    (5120, 13824, 768, [768]),
    # the small shapes on which joined passes are compared with the oracle
    (256, 688, 300, [300]), (256, 688, 351, [351]), (256, 688, 1024, [1024])])
def test_how_a_prompt_is_cut(lib, d, F, tokens, passes):
    assert cut(lib, d, F, tokens) == passes


def test_every_partition_is_worth_it(lib):
    """No run of passes is joined that the times say is slower than its passes alone."""
    lib.us.restype = C.c_double
    rng = random.Random(3)
    for _ in range(200):
        d, F = rng.choice([(4096, 11008), (5120, 13824), (2048, 5504), (256, 688)])
        sh = (C.c_int * 8)(*projections(d, F))
        us = lambda rows: lib.us(sh, rows)
        tokens = rng.randint(1, 5000)
        got = cut(lib, d, F, tokens)
        assert sum(got) == tokens and all(r <= 1024 for r in got)
        alone = [256] * (tokens // 256) + [tokens % 256] * (tokens % 256 > 0)
        assert sum(map(us, got)) <= sum(map(us, alone)) + 1e-6


def test_the_shapes_of_the_gpu_test_have_odd_segments(lib):
    """The prompts of test_gpu_long_prompts.py run as one pass, and a projection of it in the tile of eight row blocks and six
    columns with so many blocks per segment and chain."""
    from tests.test_gpu_long_prompts import ODD_SEGMENTS
    want = [(23, 0), (25, 16), (35, 16)]
    for (d, F, rows), w in zip(ODD_SEGMENTS, want):
        assert cut(lib, d, F, rows) == [rows]
        pr, found = projections(d, F), []
        for KB, NB in zip(pr[::2], pr[1::2]):
            p = plan(lib, -(-rows // 32), KB, NB)
            if (p["MT"], p["CG"]) == (8, 6):
                found.append((KB // p["S"], p["chain"]))
        assert w in found, (d, F, rows, found)
