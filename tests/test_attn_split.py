"""How a batch is cut into (sequence, part) workgroups (attn_geom.h attn_split), on the CPU: every sequence has its parts once
and in order, the launch is bounded, and the even shares that the kernel takes of the device's own length cover every block."""
import ctypes as C
import os
import random
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CODE = """
#include "attn_geom.h"
extern "C" int split(int heads, int B, const int* len, unsigned* slot, int* max_parts) {
    AttnSplit s = attn_split(heads, B, len);
    for (int i = 0; i < s.n; ++i) slot[i] = s.slot[i];
    *max_parts = s.max_parts;
    return s.n;
}
"""


@pytest.fixture(scope="module")
def split(tmp_path_factory):
    d = tmp_path_factory.mktemp("split")
    (d / "split.cpp").write_text(CODE)
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-Werror", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_2503_14153_amd", "csrc"), str(d / "split.cpp"), "-o", str(d / "split.so")],
                   check=True)
    f = C.CDLL(str(d / "split.so")).split

    def call(heads, lens):
        slot, most = (C.c_uint * 64)(), C.c_int()
        n = f(heads, len(lens), (C.c_int * len(lens))(*lens), slot, C.byref(most))
        assert 1 <= n <= 64
        return [(s & 255, s >> 8 & 255, s >> 16) for s in slot[:n]], most.value
    return call


@pytest.mark.parametrize("heads", [1, 4, 12, 32, 40, 128])
def test_every_sequence_is_covered_once(split, heads):
    rng = random.Random(heads)
    for _ in range(300):
        B = rng.randint(1, 32)
        lens = [rng.choice([0, 1, 31, 32, 33, rng.randint(0, 5000), rng.randint(0, 200000)]) for _ in range(B)]
        entries, most = split(heads, lens)
        assert len(entries) <= max(B, min(64, 512 // heads))
        at = 0
        for b, n in enumerate(lens):
            own = entries[at][2]
            assert 1 <= own <= min(most, 15)
            assert entries[at: at + own] == [(b, p, own) for p in range(own)]
            at += own
            for rows in {n, n // 2, max(n - 40, 0), n + 5}:        # (the device's length; the host's is a bound)
                blocks = (rows + 31) // 32
                each = max(1, (blocks + own - 1) // own)
                assert each * own >= blocks
        assert at == len(entries) and most == max(e[2] for e in entries)


def test_the_lengths_of_the_gpu_tests_split(split):
    """The parts that the tests on the GPU say their lengths have."""
    from tests import test_gpu_appended_prompts, test_gpu_long_prompts as prompts, test_gpu_ragged_attention as steps

    def parts(heads, lens):
        return [own for _, part, own in split(heads, lens)[0] if part == 0]
    assert [max(parts(heads, old)) for heads, old in prompts.RAGGED] == [1, 6, 15]
    assert [max(parts(32, lens)) for lens in steps.LENGTHS] == [3, 1, 3]
    assert [parts(4, lens) for lens in steps.MANY_PARTS] == [[15, 1], [15, 10, 1]]
    assert set(parts(32, test_gpu_appended_prompts.OLD)) == {1}
