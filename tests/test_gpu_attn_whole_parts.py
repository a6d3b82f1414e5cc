"""Trees of 33 to 64 nodes whose (sequence, head, row block) is cut into three or four parts of one row block each."""
import ctypes as C
import dataclasses

import pytest

import workload as wl
from tests.test_gpu_configs import _run_batch_steps

# (heads, head_dim, nodes, committed rows, parts): a first part that is not full, rows that end inside, at and just past a cache
# block, a last part that has hardly more than the tree's blocks, the longest cache that is cut so
CASES = [(32, 128, 64, 513, 4), (32, 64, 33, 700, 4), (40, 128, 50, 700, 3), (32, 128, 40, 1024, 4), (32, 64, 64, 1025, 4), (32, 64, 40, 4150, 4)]
# (heads, head_dim, nodes, committed rows of each sequence, parts): the parts come from the longest, the others' blocks are dealt to
# as many, some of which then have none
RAGGED = [(16, 64, 40, [1500, 96], 4), (13, 64, 64, [33, 700, 1024], 3), (8, 64, 33, [900, 5, 512, 64], 4), (20, 128, 64, [31, 1000], 3)]


def test_the_cases_are_cut_so(tmp_path):
    import os
    import subprocess
    from tests.test_attn_geometry import ROOT
    (tmp_path / "g.cpp").write_text('#include "attn_geom.h"\nextern "C" int parts(int h, int B, int Tp, int n) { return attn_whole_parts(h, B, Tp, n); }\n')
    subprocess.run(["g++", "-std=c++17", "-shared", "-fPIC", "-I", os.path.join(ROOT, "paper_2503_14153_amd", "csrc"),
                    str(tmp_path / "g.cpp"), "-o", str(tmp_path / "g.so")], check=True)
    parts = C.CDLL(str(tmp_path / "g.so")).parts
    for heads, _, _, rows, P in CASES:
        assert parts(heads, 1, 64, rows) == P
    for heads, _, _, rows, P in RAGGED:
        assert parts(heads, len(rows), 64, max(rows)) == P
    assert parts(32, 1, 64, 300) == 1 and parts(32, 1, 64, 5000) == 0 and parts(4, 1, 64, 1000) == 0 and parts(32, 2, 64, 2000) == 0
    assert parts(32, 1, 128, 3000) == 0 and parts(32, 1, 32, 1000) == 0
    # all workgroups of a (sequence, head) are on one XCD: none of the eight has more of them than its 32 compute units
    seen = set()
    for heads in range(1, 65):
        for B in range(1, 5):
            for rows in range(1, 5000, 31):
                P = parts(heads, B, 64, rows)
                assert P in (0, 1, 3, 4)
                if P > 1:
                    assert -(-heads * B // 8) * 2 * P <= 32
                    seen.add((heads * B, P))
    assert seen == {(32, 4)} | {(pairs, 3) for pairs in range(33, 41)}


@pytest.mark.gpu
@pytest.mark.parametrize("heads,hd,T,rows,P", CASES)
def test_parts_of_one_row_block(heads, hd, T, rows, P):
    import paper_2503_14153_amd as sd
    shape = dataclasses.replace(wl.preset("tiny").model, dtype="bf16", n_heads=heads, head_dim=hd, d_model=heads * hd, d_ffn=256,
                                n_medusa=5, topk=8, vocab=1000)
    print(_run_batch_steps(sd, shape, 1, T, [rows], rows + 60, n_steps=2))


@pytest.mark.gpu
@pytest.mark.parametrize("heads,hd,T,rows,P", RAGGED)
def test_parts_of_a_ragged_batch(heads, hd, T, rows, P):
    import paper_2503_14153_amd as sd
    shape = dataclasses.replace(wl.preset("tiny").model, dtype="bf16", n_heads=heads, head_dim=hd, d_model=heads * hd, d_ffn=256,
                                n_medusa=5, topk=8, vocab=1000)
    print(_run_batch_steps(sd, shape, len(rows), T, rows, max(rows) + 60, n_steps=2))
