"""Prompt passes in k_gemm_tile: the gate/up projection that leaves silu(gate) * up as the next operand, and the tile of eight by
eight blocks that folds its sums away between chains of products."""
import ctypes as C
import dataclasses
import os
import subprocess

import pytest
import torch

import workload as wl
from tests.test_gpu_long_prompts import _check, sd  # noqa: F401  (sd: the fixture)
from tests.test_prompt_plans import cut, lib as all_plans  # noqa: F401  (all_plans: the fixture)

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CODE = """
#include "gemm_plan.h"
extern "C" void plan(int MB, int KB, int NB, int gate_up, int* out) {
    GemmPlan p;
    double cycles;
    gemm_plan_prompt(&p, MB, KB, NB, &cycles, gate_up);
    int v[] = {gemm_plan_swiglu(p), p.chain, p.MT, p.CG, p.S, gemm_chain_limit(KB, NB)};
    for (int i = 0; i < 6; ++i) out[i] = v[i];
}
"""

# (d_model, d_ffn, rows): sums in chains of 8 and 4 blocks, d_ffn half a column block over, a last group of two pairs; 25 row blocks
# (the last tile has one) and 15 pairs of column blocks; 16 row blocks, a last group of two pairs
SWIGLU = [(192, 1616, 1000), (64, 720, 800), (64, 944, 512)]

# (d_model, d_ffn, rows), eight by eight blocks in chains of 16, 16 and 4: a last tile of two row blocks, the second of 13 rows, and a
# last group of two columns
FOLDED = (576, 7712, 557)

# (d_model, head_dim, d_ffn, rows), the down projection in eight by eight blocks, four segments: chains of 64, 64 and 44; 32, 32 and 31, a
# last tile of three row blocks and a last group of two columns
SEGMENTS = [(4096, 128, 11008, 1024), (3904, 64, 6080, 589)]


@pytest.fixture(scope="module")
def plan(tmp_path_factory, all_plans):
    d = tmp_path_factory.mktemp("tiles")
    (d / "p.cpp").write_text(CODE)
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-I", os.path.join(ROOT, "paper_2503_14153_amd", "csrc"),
                    str(d / "p.cpp"), "-o", str(d / "p.so")], check=True)
    lib = C.CDLL(str(d / "p.so"))

    def call(rows, KB, NB, gate_up):
        out = (C.c_int * 6)()
        lib.plan(-(-rows // 32), KB, NB, gate_up, out)
        return dict(zip(["swiglu", "chain", "MT", "CG", "S", "limit"], out))
    call.cut = lambda d, F, tokens: cut(all_plans, d, F, tokens)
    return call


def test_the_shapes_below_take_those_paths(plan):
    got = [plan(rows, d // 16, 2 * -(-F // 32), 1) for d, F, rows in SWIGLU]
    assert all(p["swiglu"] for p in got) and [p["chain"] for p in got] == [8, 0, 0]
    assert plan(1024, 256, 688, 1)["swiglu"] and plan(1024, 256, 688, 1)["chain"] == 128
    d, F, rows = FOLDED
    p = plan(rows, d // 16, 2 * -(-F // 32), 1)
    assert (p["MT"], p["CG"], p["S"], p["chain"]) == (8, 8, 1, 16) and d // 16 == 36 and 2 * -(-F // 32) % 8 == 2
    for (d, _, F, rows), (n, chain) in zip(SEGMENTS, [(172, 64), (95, 32)]):
        p = plan(rows, F // 16, d // 32, 0)
        assert (p["MT"], p["CG"], p["S"], p["chain"]) == (8, 8, 4, chain) and F // 16 == 4 * n
    # (and each prompt is one pass)
    for d, F, rows in [FOLDED] + [(d, F, rows) for d, _, F, rows in SEGMENTS]:
        assert plan.cut(d, F, rows) == [rows]


def test_chains_in_tiles_of_eight_by_eight_are_no_longer_than_in_a_256_row_pass(plan):
    seen = 0
    for KB, NB in [(688, 128), (320, 480), (320, 864), (864, 160), (1000, 128), (512, 512), (2048, 256)]:
        for rows in range(288, 1025, 32):
            p = plan(rows, KB, NB, 0)
            n = KB // p["S"]
            assert KB % p["S"] == 0 and (p["chain"] or n <= max(p["limit"], 8))
            if not p["chain"] or (p["MT"], p["CG"]) != (8, 8):
                continue
            seen += 1
            assert p["chain"] % 8 == 0 and 0 < p["chain"] <= max(p["limit"], 8) and p["chain"] < n
    assert seen > 20


@pytest.mark.gpu
@pytest.mark.parametrize("d,d_ffn,rows", SWIGLU)
def test_gate_up_that_leaves_the_next_operand(sd, d, d_ffn, rows):  # noqa: F811
    _check(sd, dataclasses.replace(wl.preset("tiny").model, dtype="bf16", n_heads=d // 64, head_dim=64, d_model=d, d_ffn=d_ffn),
           [0], [rows])


@pytest.mark.gpu
def test_folded_sums_in_ragged_tiles(sd):  # noqa: F811
    d, d_ffn, rows = FOLDED
    _check(sd, dataclasses.replace(wl.preset("tiny").model, dtype="bf16", n_heads=d // 64, head_dim=64, d_model=d, d_ffn=d_ffn),
           [0], [rows])


@pytest.mark.gpu
@pytest.mark.parametrize("d,hd,d_ffn,rows", SEGMENTS)
def test_joined_segments_sum_like_single_passes(sd, d, hd, d_ffn, rows):  # noqa: F811
    """The second layer's keys and values come through the first layer's gate/up (at the 7B width, chains of 128) and down
    projection (its segments in three chains). In passes of 256 rows the same sums are taken in other orders, so the two
    float32 results differ by rounding, about 1e-6 of them, and some 1e-3 of the stored values round to a neighbour, 2^-8 away
    at most: sqrt(1e-3) * 2^-8 = 1.2e-4 of the rows' norm. A block of sums lost or added twice would be of the order of 1."""
    shape = dataclasses.replace(wl.preset("tiny").model, dtype="bf16", n_layers=2, d_model=d, n_heads=d // hd, head_dim=hd, d_ffn=d_ffn)
    model = sd.Model(shape, wl.make_weights(shape, device="cuda"), 256)
    tokens = torch.from_numpy(wl.zipf_prompt(shape.vocab, rows, seed=11)).cuda()
    got = []
    for step in (rows, 256):
        kv = sd.KVCache(model, 1, rows + 8)
        for at in range(0, rows, step):
            sd.prefill(model, kv, tokens[at:at + step].contiguous(), [min(step, rows - at)])
        got.append([t.double() for t in kv.read_rows(1, 0, 0, rows)])
    for joined, single in zip(*got):
        assert (joined - single).norm() <= 5e-4 * single.norm()
        assert (joined - single).norm(dim=(1, 2)).max() <= 5e-3 * single.norm(dim=(1, 2)).min()      # (no row by itself either)
