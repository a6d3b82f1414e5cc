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
extern "C" void plan(int MB, int KB, int NB, int* out) {
    GemmPlan p;
    double cycles;
    gemm_plan_prompt(&p, MB, KB, NB, &cycles);
    const int f[] = {p.MT, p.CG, p.S, p.RT, p.chain, p.slots_max};
    for (int i = 0; i < 6; ++i) out[i] = f[i];
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


def plan(lib, MB, KB, NB):
    out = (C.c_int * 6)()
    lib.plan(MB, KB, NB, out)
    return dict(zip(["MT", "CG", "S", "RT", "chain", "slots"], out))


def shapes():
    """(d_model, d_ffn) -> the four projections in blocks of 16 inputs and 32 outputs."""
    rng = random.Random(5)
    for d, F in [(4096, 11008), (5120, 13824), (256, 688), (64, 16)] + [(32 * rng.randint(1, 256), 16 * rng.randint(1, 1800)) for _ in range(60)]:
        gu = 2 * (-(-F // 32))
        yield from [(d // 16, 3 * d // 32), (d // 16, d // 32), (d // 16, gu), (F // 16, d // 32)]


def test_chains_are_no_longer_than_in_a_256_row_pass(lib):
    folds = 0
    for KB, NB in shapes():
        limit = lib.limit(KB, NB)
        for MB in range(9, 33):
            p = plan(lib, MB, KB, NB)
            n, chain = KB // p["S"], p["chain"]
            assert KB % p["S"] == 0 and p["slots"] == p["S"] and p["MT"] * p["RT"] >= MB
            assert min(n, chain or n) <= max(limit, 8), (KB, NB, MB, p, limit)
            if chain:
                folds += 1
                assert chain % 8 == 0 and chain < n            # (the kernels' grain; there is something to fold)
                assert p["MT"] * p["CG"] <= 32 or (p["MT"], p["CG"]) == (8, 6)
    assert folds > 100
