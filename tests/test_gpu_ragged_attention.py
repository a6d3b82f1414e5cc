"""Ragged batches of one query block whose sequences are cut into parts by their lengths, or have one each: the logits are those of
each sequence decoded alone (another split of the same sums), at lengths around the parts' and blocks' edges."""
import dataclasses

import numpy as np
import pytest
import torch

import workload as wl
from tests.test_gpu_configs import _run_batch_steps

pytestmark = pytest.mark.gpu


# three parts for the longest, one each, three (test_attn_split.py has the numbers)
LENGTHS = [[600, 1, 31, 32, 33, 64], [256, 65, 0, 95, 96, 97], [1000, 10, 10, 10, 10, 2]]
# few heads: fifteen parts beside one; fifteen, ten and one
MANY_PARTS = [[5000, 100], [4600, 2400, 33]]


@pytest.mark.parametrize("T", [1, 7, 32])
@pytest.mark.parametrize("lens", LENGTHS)
def test_even_parts_of_a_ragged_batch(T, lens):
    """Reference: the same rows and drafts in a batch of one (float32 sums in another order, keys and values of the step
    rounded to bfloat16 on both sides: bound 2e-3 relative, as a flipped rounding gives)."""
    import paper_2503_14153_amd as sd
    shape = dataclasses.replace(wl.preset("tiny").model, dtype="bf16", n_heads=32, head_dim=128, d_model=4096, d_ffn=256)
    weights = {k: v.cuda() for k, v in wl.make_weights(shape, device="cuda").items()}
    model = sd.Model(shape, weights, 256)
    B, cap = len(lens), max(lens) + 8                      # 6 x 32 heads: one workgroup per (sequence, head)
    kvs = [sd.KVCache(model, B, cap)] + [sd.KVCache(model, 1, cap) for _ in lens]
    g = np.random.default_rng(8)
    root, cand = g.integers(shape.vocab, size=B), g.integers(shape.vocab, size=(B, shape.n_medusa, shape.topk))
    for b, n in enumerate(lens):
        for layer in range(shape.n_layers):
            if n:
                k, v = (wl.synthetic_kv_rows(3, f"{t}{b}.{layer}", (n, 32, 128), "bf16", "cuda") for t in "kv")
                kvs[0].write_rows(layer, b, 0, k, v)
                kvs[1 + b].write_rows(layer, 0, 0, k, v)
        kvs[1 + b].set_len([n])
        kvs[1 + b].set_draft([root[b]], cand[b: b + 1])
    kvs[0].set_len(lens)
    kvs[0].set_draft(root, cand)
    words = torch.zeros((shape.vocab + 31) // 32, dtype=torch.int32, device="cuda")
    tree = sd.Tree(*wl.default_tree(T, shape.n_medusa, shape.topk), shape.n_medusa, shape.topk)
    got = sd.spec_step(model, kvs[0], tree, words, want_logits=True).logits
    for b in range(B):
        want = sd.spec_step(model, kvs[1 + b], tree, words, want_logits=True).logits[0]
        assert torch.isfinite(got[b]).all()
        assert float((got[b] - want).norm() / want.norm()) < 2e-3


# one row each: merged by the O projection, or (three sequences) by the launch for a handful of rows; 14, 21 and more by the other
@pytest.mark.parametrize("T", [1, 7, 30])
@pytest.mark.parametrize("lens", MANY_PARTS)
def test_many_parts_against_the_oracle(T, lens):
    import paper_2503_14153_amd as sd
    shape = dataclasses.replace(wl.preset("tiny").model, dtype="bf16")
    rep = _run_batch_steps(sd, shape, len(lens), T, lens, max(lens) + 40, n_steps=2)
    print(f"\n[tiny {lens} T={T}] {rep}")
