"""Passes whose sequences do not fill 32-row blocks: the rows of a pass are packed without padding between sequences, and a
prompt pass holds only the sequences that still have tokens. Reference: the oracle, sequence by sequence."""
import dataclasses

import numpy as np
import pytest
import torch

import workload as wl
from oracle import specdec_oracle as orc
from tests import lockstep

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sd():
    import paper_2503_14153_amd as sd
    sd.lib()
    return sd


@pytest.fixture(scope="module")
def tiny(sd):
    shape = dataclasses.replace(wl.preset("tiny").model, dtype="bf16")
    weights = wl.make_weights(shape, medusa_bias_std=0.1)
    return shape, {k: v.cuda() for k, v in weights.items()}, lockstep.weights_to_f64(weights)


@pytest.mark.parametrize("B,T", [(1, 1), (8, 1), (3, 1), (5, 12), (2, 31), (4, 33), (3, 40), (2, 65), (8, 32)])
def test_ragged_prompts_and_packed_steps_match_the_oracle(sd, tiny, B, T):
    """Ragged prompts (some end passes before others, one is a single token), then two steps: row counts of B * T on both
    sides of 8-row groups, row blocks and powers of two of them; every sequence against its own oracle run."""
    shape, weights, w64 = tiny
    cap = 400
    model = sd.Model(shape, weights, 256)
    kv = sd.KVCache(model, B, cap)
    lens = [300, 1, 97, 40, 64, 5, 33, 128][:B]
    prompts = [wl.zipf_prompt(shape.vocab, n, seed=50 + b) for b, n in enumerate(lens)]
    stop = wl.stop_set(shape.vocab, 0.2)
    words = torch.from_numpy(wl.pack_mask_words(stop).view(np.int32)).cuda()
    sd.prefill(model, kv, torch.from_numpy(np.concatenate(prompts)).cuda(), lens)
    assert kv.len() == lens
    rep = lockstep.Report()
    sts = [orc.prefill(w64, shape, p, cap) for p in prompts]
    for b, st in enumerate(sts):
        lockstep.compare_kv_rows(kv, st, shape, 0, lens[b], rep, seq=b)
        lockstep.check_cand(kv.get_draft()[1][b].cpu().numpy(), st.cand, orc.medusa_logits(w64, shape, _h_last(w64, shape, prompts[b])), rep)
    tree_np = wl.default_tree(T, shape.n_medusa, shape.topk)
    tree = sd.Tree(*tree_np, shape.n_medusa, shape.topk)
    for _ in range(2):
        for b, st in enumerate(sts):                       # both sides start from the oracle's history and drafts
            lockstep.resync_kv_rows(kv, st, shape, max(st.kv.n - 8, 0), seq=b)
        kv.set_len([st.kv.n for st in sts])
        kv.set_draft([st.root_tok for st in sts], np.stack([st.cand for st in sts]))
        n_old = [st.kv.n for st in sts]
        if T == 1:
            out = sd.greedy_step(model, kv, want_logits=True, want_head_logits=True)
        else:
            out = sd.spec_step(model, kv, tree, words, want_logits=True, want_argmax=True, want_head_logits=True)
        torch.cuda.synchronize()
        now = kv.len()
        for b, st in enumerate(sts):
            if T == 1:
                rec = orc.greedy_step(w64, shape, st)
                lockstep.check_logits(out.logits[b].cpu().numpy().astype(np.float64), rec.logits, rep)
                n_acc, same = 1, True
                assert int(out.tokens[b, 0]) == int(rec.tokens[0])
            else:
                rec = orc.spec_step(w64, shape, st, tree_np, stop, "keep_all")
                n_acc, chain = lockstep.check_step_outputs(out, b, rec, tree_np, stop, "keep_all", shape, rep)
                same = n_acc == rec.n_accept and chain[:n_acc] == list(rec.src_slots)
            assert now[b] == n_old[b] + n_acc
            if same:
                lockstep.compare_kv_rows(kv, st, shape, n_old[b], n_old[b] + n_acc, rep, seq=b)
                err = np.abs(out.head_logits[b].cpu().numpy().astype(np.float64) - rec.head_logits).max()
                assert err <= 2 * lockstep.LOGIT_MAX_ABS
    # rows of the last prompt pass stay committable, also where it held only some of the sequences
    kv.set_len([0] * B)
    sd.prefill(model, kv, torch.from_numpy(np.concatenate(prompts)).cuda(), lens)
    slots = torch.zeros((B, 2), dtype=torch.int32, device="cuda")
    count = torch.tensor([2] + [0] * (B - 1), dtype=torch.int32, device="cuda")      # sequence 0 ends last
    sd.kv_commit_rows(model, kv, slots, count)
    assert kv.len() == [lens[0] + 2] + lens[1:]
    k, v = kv.read_rows(shape.n_layers - 1, 0, lens[0], 2)
    assert torch.equal(k[0], k[1]) and torch.equal(v[0], v[1])
    k0, v0 = kv.read_rows(shape.n_layers - 1, 0, 0, lens[0])
    assert any(torch.equal(k[0], k0[j]) and torch.equal(v[0], v0[j]) for j in range(lens[0]))


def _h_last(w64, shape, prompt):
    n = len(prompt)
    kv = orc.KVCache.empty(shape, n)
    return orc.forward_rows(w64, shape, prompt, np.arange(n), np.tril(np.ones((n, n), bool)), kv)[1][-1]
