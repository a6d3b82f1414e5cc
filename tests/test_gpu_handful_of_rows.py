"""Passes of a handful of rows, whose projections finish every column in one workgroup: at the edges of what takes that path
(8 rows of the layers, 16 of the LM head; up to 32 the contraction is dealt to the waves too), with a contraction that ends in half a step (d_ffn = 43 * 16), against the oracle."""
import dataclasses

import pytest
import torch

import workload as wl
from tests.test_gpu_configs import _run_batch_steps

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sd():
    import paper_2503_14153_amd as sd
    sd.lib()
    return sd


# three heads: the base and head rows of plain decoding are 4 B (16 for B = 4, 20 for B = 5), a tree's head rows 3 B
@pytest.mark.parametrize("B,T", [(1, 1), (2, 1), (3, 1), (4, 1), (5, 1), (8, 1), (3, 3), (1, 3), (1, 8), (1, 9), (2, 4), (1, 16), (6, 3), (1, 17), (2, 16), (1, 33)])
def test_a_handful_of_rows_against_the_oracle(sd, B, T):
    shape = dataclasses.replace(wl.preset("tiny").model, dtype="bf16", vocab=1000 + 17 * (B == 3))
    rep = _run_batch_steps(sd, shape, B, T, [40 + 13 * b for b in range(B)], 200, n_steps=2)
    print(f"\n[tiny B={B} T={T}] {rep}")


# the widest model whose O projection merges the attention parts in LDS (8 bytes an input, 65.5 KiB with the sums'), and the next
@pytest.mark.parametrize("heads", [96, 97])
@pytest.mark.parametrize("B", [1, 2])
def test_one_and_two_rows_at_the_widest(sd, B, heads):
    shape = dataclasses.replace(wl.preset("tiny").model, dtype="bf16", n_layers=1, n_heads=heads, head_dim=64, d_model=64 * heads, d_ffn=256)
    rep = _run_batch_steps(sd, shape, B, 1, [100, 33][:B], 120, n_steps=2, weights_device="cuda")
    print(f"\n[{heads} heads B={B}] {rep}")


@pytest.mark.parametrize("B", [1, 3, 8])
def test_with_and_without_draft_heads(sd, B):
    """The base logits of plain decoding do not depend on whether the head rows share their pass of the LM head (bit for bit
    while all of them take the same path: 4 rows; beyond that to float32 sums of 256 products of two 16-bit terms)."""
    shape = dataclasses.replace(wl.preset("tiny").model, dtype="bf16")
    weights = wl.make_weights(shape, medusa_bias_std=0.1)
    model = sd.Model(shape, {k: v.cuda() for k, v in weights.items()}, 256)
    kv = sd.KVCache(model, B, 100)
    lens = [20 + b for b in range(B)]
    sd.prefill(model, kv, torch.from_numpy(wl.zipf_prompt(shape.vocab, sum(lens))).cuda(), lens)
    root, cand = (t.clone() for t in kv.get_draft())
    a = sd.greedy_step(model, kv, want_logits=True)
    kv.set_len(lens)
    kv.set_draft(root, cand)
    model.set_greedy_drafts(False)
    b = sd.greedy_step(model, kv, want_logits=True)
    if B == 1:
        assert torch.equal(a.logits, b.logits)
    # two terms keep each operand to 2^-17 of itself, and float32 sums of 256 terms to 256 * 2^-24 of theirs
    tol = (2 ** -16 + 256 * 2.0 ** -24) * 256 ** 0.5
    assert float((a.logits - b.logits).abs().max()) <= tol * float(a.logits.abs().max())
