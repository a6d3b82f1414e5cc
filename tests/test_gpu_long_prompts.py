"""Prompts of more than 256 rows: several chunks of every sequence run as one pass whose rows are committed layer by layer.
Committed rows, root and candidates against the oracle, and the rows that a commit afterwards finds."""
import dataclasses

import numpy as np
import pytest
import torch

import workload as wl
from oracle import specdec_oracle as orc
from tests import lockstep
from tests.test_gpu_configs import _fill_synthetic

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sd():
    import paper_2503_14153_amd as sd
    sd.lib()
    return sd


# one chunk and a remainder, a last tile that is nearly empty, two passes of 1024 rows and a remainder that starts inside a cache
# block, ragged batches (chunks of 64 rows joined up to 256; prompts that end in the middle of the pass), two passes that fit 256 rows together
@pytest.mark.parametrize("old,new", [([0], [300]), ([0], [351]), ([37], [1100]), ([2, 5, 33], [700, 40, 300]),
                                     ([1, 6, 64, 31], [90, 400, 129, 64]), ([9, 3], [100, 150])])
def test_long_prompts_against_the_oracle(sd, old, new):
    _check(sd, dataclasses.replace(wl.preset("tiny").model, dtype="bf16"), old, new)


# committed rows: one part each, one sequence of six parts, one of fifteen (test_attn_split.py has the numbers)
RAGGED = [(32, [300, 5, 64, 31, 40, 1, 33, 90]), (32, [1300, 5, 64, 31, 40, 1, 33, 90]), (4, [5000, 5, 700, 31, 40, 1, 33, 90])]


@pytest.mark.parametrize("heads,old", RAGGED)
def test_a_ragged_batch_in_one_pass(sd, heads, old):
    """Eight sequences, one pass of at most 32 rows each: attention with as many parts as each sequence's rows ask for."""
    _check(sd, dataclasses.replace(wl.preset("tiny").model, dtype="bf16", n_heads=heads, head_dim=64, d_model=64 * heads, d_ffn=256),
           old, [20, 32, 1, 7, 25, 31, 3, 12])


# a projection in k_gemm_tile whose segments have an odd number of contraction blocks (the kernel takes them in pairs): 23 in one
# chain, 25 in chains of 16 and 9, 35 in 16, 16 and 3 with a last column group of four blocks (test_prompt_plans.py has the numbers)
ODD_SEGMENTS = [(1472, 2768, 400), (1600, 2768, 300), (2240, 400, 1010)]


@pytest.mark.parametrize("d,d_ffn,rows", ODD_SEGMENTS)
def test_segments_of_an_odd_number_of_blocks(sd, d, d_ffn, rows):
    _check(sd, dataclasses.replace(wl.preset("tiny").model, dtype="bf16", n_heads=d // 64, head_dim=64, d_model=d, d_ffn=d_ffn),
           [0], [rows])


# one to eight rows in a pass whose row blocks are those of the widest (padded) pass: alone, behind committed rows, and the
# remainder of a prompt of whole passes
@pytest.mark.parametrize("old,new", [([0], [5]), ([100], [8]), ([40], [1]), ([0], [1024 + 3]), ([7, 70], [2, 6])])
def test_prompts_that_end_in_a_handful_of_rows(sd, old, new):
    _check(sd, dataclasses.replace(wl.preset("tiny").model, dtype="bf16", n_heads=32, head_dim=64, d_model=2048, d_ffn=256), old, new)


# QKV at the 7B and the 13B width: four and two chains in one segment of the joined pass, four and two segments of a 256-row pass
@pytest.mark.parametrize("d,heads,d_ffn,rows", [(4096, 32, 11008, 1024), (5120, 40, 13824, 768)])
def test_a_joined_pass_sums_like_single_ones(sd, d, heads, d_ffn, rows):
    """One layer's keys and values depend on the QKV projection alone. The joined pass cuts its contraction into chains as long as
    a 256-row pass's segments, added in the same order, so that the cache rows of a prompt are the same bits whether it comes in
    one call or in calls of 256 tokens: no float32 sum is longer for the joining. (One chain over the whole contraction was 4.5 %
    further from 64 bits; this showed in one of 400 stored values.)"""
    shape = dataclasses.replace(wl.preset("tiny").model, dtype="bf16", n_layers=1, d_model=d, n_heads=heads, head_dim=128, d_ffn=d_ffn)
    model = sd.Model(shape, wl.make_weights(shape, device="cuda"), 256)
    tokens = torch.from_numpy(wl.zipf_prompt(shape.vocab, rows, seed=7)).cuda()
    got = []
    for step in (rows, 256):
        kv = sd.KVCache(model, 1, rows + 8)
        for at in range(0, rows, step):
            sd.prefill(model, kv, tokens[at:at + step].contiguous(), [step])
        got.append(kv.read_rows(0, 0, 0, rows))
    assert got[0][0].float().std() > 0.1
    for joined, single in zip(*got):
        assert torch.equal(joined, single)


def _check(sd, shape, old, new):
    weights = wl.make_weights(shape, medusa_bias_std=0.1)
    w64 = lockstep.weights_to_f64(weights)
    model = sd.Model(shape, {k: v.cuda() for k, v in weights.items()}, 256)
    B, cap = len(old), max(a + n for a, n in zip(old, new)) + 40
    kv = sd.KVCache(model, B, cap)
    states = [orc.DecodeState(orc.KVCache.empty(shape, cap)) for _ in old]
    if any(old):
        _fill_synthetic(kv, states, shape, old)
    prompts = [wl.zipf_prompt(shape.vocab, n, seed=90 + b) for b, n in enumerate(new)]
    sd.prefill(model, kv, torch.from_numpy(np.concatenate(prompts)).cuda(), new)
    total = [a + n for a, n in zip(old, new)]
    assert kv.len() == total
    root, cand = (t.cpu().numpy() for t in kv.get_draft())
    rep = lockstep.Report()
    for b, st in enumerate(states):
        n = new[b]
        logits, h, k, v = orc.forward_rows(w64, shape, prompts[b], old[b] + np.arange(n), np.tril(np.ones((n, n), bool)), st.kv)
        st.kv.k[:, old[b]:total[b]], st.kv.v[:, old[b]:total[b]] = k, v
        lockstep.compare_kv_rows(kv, st, shape, 0, total[b], rep, seq=b)
        gap = logits[-1].max() - logits[-1][root[b]]
        assert gap < lockstep.NEAR_TIE, f"sequence {b}: root {root[b]} lies {gap:.3g} below the oracle's"
        lockstep.check_cand(cand[b], orc.medusa_candidates(w64, shape, h[-1]), orc.medusa_logits(w64, shape, h[-1]), rep)
    # the last pass by itself held max_rows / (prompts still running) rows of each, in multiples of 32
    left, start = list(new), list(old)
    while True:
        running = [b for b in range(B) if left[b] > 0]
        tp = 256 // len(running) // 32 * 32
        took = {b: min(left[b], tp) for b in running}
        if all(left[b] <= tp for b in running):
            break
        for b, n in took.items():
            left[b] -= n
            start[b] += n
    slots = [0, max(took.values()) // 2, max(took.values()) - 1]
    sd.kv_commit_rows(model, kv, torch.tensor([slots] * B, dtype=torch.int32, device="cuda"),
                      torch.tensor([3] * B, dtype=torch.int32, device="cuda"))
    assert kv.len() == [total[b] + (3 if b in took else 0) for b in range(B)]
    for b, n in took.items():
        for layer in range(shape.n_layers):
            for got, have in zip(kv.read_rows(layer, b, total[b], 3), kv.read_rows(layer, b, 0, total[b])):
                for j, s in enumerate(slots):
                    assert torch.equal(got[j], have[start[b] + min(s, n - 1)]), f"sequence {b}, layer {layer}, slot {s}"
