"""Prompts appended to ragged caches, and steps of one and two rows at the widths where the projections build their own
operands, against the oracle."""
import dataclasses

import numpy as np
import pytest
import torch

import workload as wl
from oracle import specdec_oracle as orc
from tests import lockstep
from tests.test_gpu_configs import _fill_synthetic, _run_batch_steps

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sd():
    import paper_2503_14153_amd as sd
    sd.lib()
    return sd


OLD = [300, 5, 64, 31, 40, 1, 33, 90]


def test_prompts_appended_to_a_ragged_batch(sd):
    """Eight sequences of 32 heads (one workgroup per (sequence, head)) whose caches hold 1 to 300 rows get 1 to 45 more
    tokens each: rows packed without padding, attention in one part per sequence; the longest prompt needs a
    pass of its own. Committed rows, root and candidates of every sequence against its own oracle run."""
    shape = dataclasses.replace(wl.preset("tiny").model, dtype="bf16", n_heads=32, head_dim=64, d_model=2048, d_ffn=256)
    weights = wl.make_weights(shape, medusa_bias_std=0.1)
    w64 = lockstep.weights_to_f64(weights)
    model = sd.Model(shape, {k: v.cuda() for k, v in weights.items()}, 256)
    old, new, cap = OLD, [20, 32, 1, 7, 45, 31, 3, 12], 340
    kv = sd.KVCache(model, 8, cap)
    states = [orc.DecodeState(orc.KVCache.empty(shape, cap)) for _ in old]
    _fill_synthetic(kv, states, shape, old)
    prompts = [wl.zipf_prompt(shape.vocab, n, seed=70 + b) for b, n in enumerate(new)]
    sd.prefill(model, kv, torch.from_numpy(np.concatenate(prompts)).cuda(), new)
    assert kv.len() == [a + n for a, n in zip(old, new)]
    root, cand = (t.cpu().numpy() for t in kv.get_draft())
    rep = lockstep.Report()
    for b, st in enumerate(states):
        n = new[b]
        logits, h, k, v = orc.forward_rows(w64, shape, prompts[b], old[b] + np.arange(n), np.tril(np.ones((n, n), bool)), st.kv)
        st.kv.k[:, old[b]:old[b] + n], st.kv.v[:, old[b]:old[b] + n] = k, v
        lockstep.compare_kv_rows(kv, st, shape, 0, old[b] + n, rep, seq=b)
        gap = logits[-1].max() - logits[-1][root[b]]
        assert gap < lockstep.NEAR_TIE, f"sequence {b}: root {root[b]} lies {gap:.3g} below the oracle's"
        heads = orc.medusa_logits(w64, shape, h[-1])
        lockstep.check_cand(cand[b], orc.medusa_candidates(w64, shape, h[-1]), heads, rep)


@pytest.mark.parametrize("B,T", [(1, 1), (2, 1), (1, 2)])
def test_steps_of_one_and_two_rows_against_the_oracle(sd, B, T):
    shape = dataclasses.replace(wl.preset("7b", 1).model, dtype="bf16", vocab=1000)
    rep = _run_batch_steps(sd, shape, B, T, [300, 33][:B], 320, n_steps=2, weights_device="cuda")
    print(f"\n[7b L1 B={B} T={T}] {rep}")
