"""How a pass's attention is cut into parts (attn_geom.h), on the CPU over every length: a captured step is replayed wherever
the geometry is the one it was captured with, so an equal geometry has to mean that every committed block is covered."""
import ctypes as C
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CODE = """
#include "attn_geom.h"
extern "C" void geometry(int fused, int heads, int parts, int B, int Tp, int n_hi, int ragged, int* out) {
    AttnGeom g = attn_geometry_of_pass(fused != 0, heads, parts, B, Tp, n_hi, ragged != 0);
    out[0] = g.ncparts; out[1] = g.per; out[2] = g.tree_sep; out[3] = g.nparts;
}
extern "C" int whole(int heads, int B, int Tp, int n_hi) { return attn_whole_pays(heads, B, Tp, n_hi); }
"""


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    d = tmp_path_factory.mktemp("geom")
    (d / "geom.cpp").write_text(CODE)
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_2503_14153_amd", "csrc"), str(d / "geom.cpp"), "-o", str(d / "geom.so")],
                   check=True)
    return C.CDLL(str(d / "geom.so"))


@pytest.fixture(scope="module")
def geometry(lib):
    out = (C.c_int * 4)()

    def call(*a):
        lib.geometry(*a, out)
        return tuple(out)
    return call


@pytest.mark.parametrize("ragged", [0, 1])
@pytest.mark.parametrize("fused", [0, 1])
@pytest.mark.parametrize("heads", [1, 4, 32, 40])
@pytest.mark.parametrize("B,Tp", [(1, 32), (1, 64), (1, 128), (1, 256), (2, 32), (4, 64), (5, 32), (8, 32)])
def test_every_committed_block_is_covered(geometry, heads, B, Tp, fused, ragged):
    launched = {}
    for n_hi in range(0, 20001, 32 if B > 1 else 1):
        nblk = (n_hi + 31) // 32
        g = geometry(fused, heads, 65, B, Tp, n_hi, ragged)
        ncparts, per, tree_sep, nparts = g
        assert nparts == ncparts + tree_sep and 1 <= nparts <= 65 and per >= 0
        launched.setdefault(g, []).append(nblk)
        if per == 0:                                       # parts that take their shares from the device's own lengths
            assert not fused and ragged and Tp == 32 and ncparts == 2
            continue
        assert ncparts * per >= nblk and (ncparts == 0 or (ncparts - 1) * per < nblk)
        if fused:
            assert tree_sep <= 1                           # its attention launch does not build the tree's keys
    for (ncparts, per, _, _), blocks in launched.items():
        assert per == 0 or max(blocks) <= ncparts * per


# both sides of the line as measured (attn_geom.h): one round of workgroups by the blocks each has, a second round dearer
@pytest.mark.parametrize("heads,B,Tp,n_hi,pays", [
    (32, 1, 64, 300, 1), (32, 1, 64, 700, 0), (32, 1, 32, 300, 0), (32, 1, 256, 1700, 1), (32, 1, 256, 5000, 0), (4, 1, 64, 300, 0),
    (40, 2, 128, 700, 1), (40, 2, 128, 2000, 0), (40, 1, 256, 500, 1), (40, 1, 256, 2250, 0), (40, 4, 64, 100, 0), (40, 4, 64, 1000, 0),
    (40, 3, 64, 1000, 1)])
def test_where_one_workgroup_per_row_block_pays(lib, heads, B, Tp, n_hi, pays):
    assert lib.whole(heads, B, Tp, n_hi) == pays
