"""Captured steps: what a replay may not carry over from the moment of its capture. Reference: the same steps eager, bit for
bit (the kernels are deterministic)."""
import dataclasses

import numpy as np
import pytest
import torch

import workload as wl

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def sd():
    import paper_2503_14153_amd as sd
    sd.lib()
    return sd

@pytest.mark.parametrize("T", [1, 16])
def test_float32_steps_replay(sd, T):
    """The float32 path has no attention parts to key a graph by: its steps are captured all the same."""
    shape = wl.preset("tiny").model
    model = sd.Model(shape, {k: v.cuda() for k, v in wl.make_weights(shape).items()}, 64)
    kv = sd.KVCache(model, 2, 128)
    words = torch.zeros((shape.vocab + 31) // 32, dtype=torch.int32, device="cuda")
    tree = sd.Tree(*wl.default_tree(T, shape.n_medusa, shape.topk), shape.n_medusa, shape.topk)
    g = np.random.default_rng(8)
    draft = g.integers(shape.vocab, size=2), g.integers(shape.vocab, size=(2, shape.n_medusa, shape.topk))
    prompt = torch.from_numpy(wl.zipf_prompt(shape.vocab, 80)).cuda()
    got = {}
    for graphs in (False, True):
        model.set_graph_mode(graphs)
        kv.set_len([0, 0])
        sd.prefill(model, kv, prompt, [70, 10])
        out, res = None, []
        for _ in range(4):                                 # the lengths grow from step to step
            kv.set_draft(*draft)
            out = sd.spec_step(model, kv, tree, words, want_logits=True, want_head_logits=True, out=out)
            torch.cuda.synchronize()
            res.append((out.logits.clone(), out.head_logits.clone(), out.tokens.clone(), kv.len()))
        got[graphs] = res
    model.set_graph_mode(False)
    for a, b in zip(got[False], got[True]):
        assert all(torch.equal(x, y) for x, y in zip(a[:3], b[:3])) and a[3] == b[3]
