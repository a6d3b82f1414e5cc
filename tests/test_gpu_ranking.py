"""Arg-max and top-k over the vocabulary, from the logits a step returns: whole numbers, so they are exactly what a stable
descending sort of those logits gives (largest first, lower id on ties)."""
import dataclasses

import numpy as np
import pytest
import torch

import workload as wl

pytestmark = pytest.mark.gpu


# vocabularies around the chunk sizes (2048, 4096, 10240 ids) and their switches (32768, 65536), multiples of four or not;
# ties = identical rows of the LM head, so equal logits, in the same thread, chunk and across chunks
@pytest.mark.parametrize("dtype,vocab,topk,B,T", [
    ("bf16", 33, 32, 1, 5), ("bf16", 1000, 4, 3, 1), ("bf16", 2049, 10, 2, 7), ("bf16", 4097, 32, 1, 33),
    ("bf16", 32768, 10, 8, 1), ("bf16", 32771, 10, 1, 16), ("bf16", 65537, 32, 2, 3), ("bf16", 131073, 8, 1, 4),
    ("f32", 33, 4, 2, 5), ("f32", 5001, 16, 1, 9)])
@pytest.mark.parametrize("tied", [False, True])
def test_argmax_and_top_k_follow_the_returned_logits(dtype, vocab, topk, B, T, tied):
    import paper_2503_14153_amd as sd
    shape = dataclasses.replace(wl.preset("tiny").model, dtype=dtype, n_layers=1, d_model=64, n_heads=1, d_ffn=64, vocab=vocab,
                                n_medusa=3, topk=topk)
    weights = wl.make_weights(shape, medusa_bias_std=0.1, std=0.1)
    if tied:                                               # many rows repeat one of a few
        g = np.random.default_rng(3)
        weights["lm_head"] = weights["lm_head"][torch.from_numpy(g.integers(0, 5, size=vocab))].contiguous()
    model = sd.Model(shape, {k: v.cuda() for k, v in weights.items()}, 256)
    kv = sd.KVCache(model, B, 64)
    g = np.random.default_rng(4)
    kv.set_draft(g.integers(vocab, size=B), g.integers(vocab, size=(B, 3, topk)))
    words = torch.zeros((vocab + 31) // 32, dtype=torch.int32, device="cuda")
    if T == 1:
        out = sd.greedy_step(model, kv, want_logits=True, want_head_logits=True)
    else:
        parent, depth, rank = wl.chain_tree(2)
        parent, depth, rank = (np.concatenate([a, x]) for a, x in
                               ((parent, np.zeros(T - 2)), (depth, np.ones(T - 2)), (rank, np.arange(1, T - 1))))
        if T - 1 > topk:                                   # siblings need distinct ranks: a second level under node 1
            n1 = topk
            parent = np.concatenate([[-1], np.zeros(n1), np.ones(T - 1 - n1)])
            depth = np.concatenate([[0], np.ones(n1), np.full(T - 1 - n1, 2)])
            rank = np.concatenate([[0], np.arange(n1), np.arange(T - 1 - n1)])
        tree = sd.Tree(parent.astype(int), depth.astype(int), rank.astype(int), 3, topk)
        out = sd.spec_step(model, kv, tree, words, want_logits=True, want_argmax=True, want_head_logits=True)
        best = out.logits.cpu().numpy().argmax(-1)         # numpy: the first maximum
        assert np.array_equal(out.argmax.cpu().numpy(), best)
    root, cand = (t.cpu().numpy() for t in kv.get_draft())
    logits, heads = out.logits.cpu().numpy(), out.head_logits.cpu().numpy()
    last = [int(s[int(n) - 1]) for s, n in zip(out.src_slots.cpu(), out.n_accept.cpu())]
    for b in range(B):
        assert root[b] == logits[b, last[b]].argmax()
        for i in range(3):
            assert np.array_equal(cand[b, i], np.argsort(-heads[b, i], kind="stable")[:topk])
