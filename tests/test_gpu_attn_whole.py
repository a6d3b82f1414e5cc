"""Trees of two to eight row blocks over few cache blocks, where one workgroup takes a (sequence, head, row block), against the
oracle: no committed rows, one, the edges of cache blocks, rows past the tree in its last block, head_dim 64 and 128."""
import dataclasses

import pytest

import workload as wl
from tests.test_gpu_configs import _run_batch_steps

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hd,B,T,lens", [(128, 1, 33, [1]), (64, 1, 64, [32]), (128, 1, 64, [300]), (64, 2, 40, [65, 480]),
                                         (64, 1, 100, [700]), (128, 1, 200, [33]), (64, 1, 256, [520])])
def test_one_workgroup_per_row_block(hd, B, T, lens):
    import paper_2503_14153_amd as sd
    shape = dataclasses.replace(wl.preset("tiny").model, dtype="bf16", n_heads=32, head_dim=hd, d_model=32 * hd, d_ffn=256, n_medusa=5,
                                topk=8, vocab=1000)
    rep = _run_batch_steps(sd, shape, B, T, lens, max(lens) + 60, n_steps=2)
    print(f"\n[hd {hd} B={B} T={T} {lens}] {rep}")
