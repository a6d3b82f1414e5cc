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


def _wide(sd, B, T, cap, max_rows):
    """32 heads over a tiny model, a cache full of known rows, random drafts."""
    shape = dataclasses.replace(wl.preset("tiny").model, dtype="bf16", n_heads=32, head_dim=128, d_model=4096, d_ffn=256)
    model = sd.Model(shape, wl.make_weights(shape, device="cuda"), max_rows)
    kv = sd.KVCache(model, B, cap)
    rows = [[[wl.synthetic_kv_rows(3, f"{t}{b}.{layer}", (cap, 32, 128), "bf16", "cuda") for t in "kv"]
             for layer in range(shape.n_layers)] for b in range(B)]
    g = np.random.default_rng(8)
    draft = g.integers(shape.vocab, size=B), g.integers(shape.vocab, size=(B, shape.n_medusa, shape.topk))
    words = torch.zeros((shape.vocab + 31) // 32, dtype=torch.int32, device="cuda")
    tree = sd.Tree(*wl.default_tree(T, shape.n_medusa, shape.topk), shape.n_medusa, shape.topk)
    return model, kv, words, tree, draft, rows


@pytest.mark.parametrize("fused", [False, True])
@pytest.mark.parametrize("B,T,lens", [
    (8, 32, [256, 288, 257, 320, 600, 256]),             # one workgroup per (sequence, head), ragged: even parts or one part
    (1, 64, [1568, 1728, 1600, 1569, 1760]),             # a tree of two blocks: in parts of its own or not
    (1, 32, [40, 41, 256, 257, 1100])])
def test_replayed_steps_follow_the_cache_length(sd, B, T, lens, fused):
    """A step captured at one length and replayed at others, in both directions across the edges of 32-row blocks: every
    committed row counts."""
    model, kv, words, tree, draft, rows = _wide(sd, B, T, max(lens) + 8, 256)
    others = [40, 1, 33, 64, 7, 100, 31][:B - 1]
    model.set_fused(fused)
    got = {}
    for graphs in (False, True):
        model.set_graph_mode(graphs)
        out, res = None, []
        for n in lens + lens:
            for b in range(B):                             # (a step overwrites the rows that it commits)
                for layer, (k, v) in enumerate(rows[b]):
                    kv.write_rows(layer, b, 0, k, v)
            kv.set_len([n] + others)
            kv.set_draft(*draft)
            out = sd.spec_step(model, kv, tree, words, want_logits=True, out=out)
            torch.cuda.synchronize()
            res.append((out.logits.clone(), out.tokens.clone(), kv.len()))
            _ = (out.logits * 2).sum().item()              # unrelated eager work between replays
        got[graphs] = res
    model.set_graph_mode(False)
    for i, (a, b) in enumerate(zip(got[False], got[True])):
        assert torch.isfinite(b[0]).all()
        assert torch.equal(a[0], b[0]), f"call {i}, length {(lens + lens)[i]}: the replay's logits are not the eager step's"
        assert torch.equal(a[1], b[1]) and a[2] == b[2]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_rows_of_a_replayed_step_can_be_committed(sd, dtype):
    """sd_kv_commit_rows after a replay takes the rows of the step that was replayed, whatever passes ran since its capture: a
    ragged prompt whose last pass held one sequence, a step of another tree."""
    shape = dataclasses.replace(wl.preset("tiny").model, dtype=dtype)
    model = sd.Model(shape, {k: v.cuda() for k, v in wl.make_weights(shape).items()}, 256)
    B, cap = 4, 160
    trees = [sd.Tree(*wl.default_tree(T, shape.n_medusa, shape.topk), shape.n_medusa, shape.topk) for T in (5, 9)]
    words = torch.zeros((shape.vocab + 31) // 32, dtype=torch.int32, device="cuda")
    lens = [100, 3, 17, 40]
    prompt = torch.from_numpy(wl.zipf_prompt(shape.vocab, sum(lens))).cuda()
    g = np.random.default_rng(8)
    draft = g.integers(shape.vocab, size=B), g.integers(shape.vocab, size=(B, shape.n_medusa, shape.topk))
    slots = torch.tensor([[0, 4], [3, 1], [2, 2], [4, 0]], dtype=torch.int32, device="cuda")
    two = torch.full((B,), 2, dtype=torch.int32, device="cuda")

    def step(kv, tree, out):
        kv.set_len(lens)
        kv.set_draft(*draft)
        return sd.spec_step(model, kv, tree, words, out=out)

    def committed(kv):
        kv.set_len(lens)
        sd.kv_commit_rows(model, kv, slots, two)
        assert kv.len() == [n + 2 for n in lens]
        return [t.clone() for b in range(B) for layer in range(shape.n_layers) for t in kv.read_rows(layer, b, lens[b], 2)]

    got = {}
    for graphs in (False, True):
        model.set_graph_mode(graphs)
        kv = sd.KVCache(model, B, cap)
        sd.prefill(model, kv, prompt, lens)
        outs, res = [None, None], []
        for i in (0, 1):
            outs[i] = step(kv, trees[i], outs[i])          # captures
        for i in (0, 1, 0):
            kv.set_len([0] * B)
            sd.prefill(model, kv, prompt, lens)
            step(kv, trees[i], outs[i])
            res.append(committed(kv))
        for i in (1, 0):                                   # and straight after the other tree's step
            step(kv, trees[i], outs[i])
            res.append(committed(kv))
        got[graphs] = res
    model.set_graph_mode(False)
    for a, b in zip(got[False], got[True]):
        assert all(torch.equal(x, y) for x, y in zip(a, b))


def test_replays_write_the_timeline_only_while_it_is_set(sd):
    """The buffer of sd_set_layer_timeline is the caller's only while it is set: a step captured with it must not be replayed
    after it was taken away, nor one captured without it while it is there."""
    shape = dataclasses.replace(wl.preset("tiny").model, dtype="bf16")
    model = sd.Model(shape, {k: v.cuda() for k, v in wl.make_weights(shape).items()}, 32)
    kv = sd.KVCache(model, 1, 128)
    words = torch.zeros((shape.vocab + 31) // 32, dtype=torch.int32, device="cuda")
    tree = sd.Tree(*wl.default_tree(16, shape.n_medusa, shape.topk), shape.n_medusa, shape.topk)
    kv.set_draft([1], np.arange(shape.n_medusa * shape.topk).reshape(1, shape.n_medusa, shape.topk))
    buf = torch.zeros((shape.n_layers + 1, 24, 256), dtype=torch.int64, device="cuda")
    model.set_fused(True)
    model.set_graph_mode(True)
    out = None
    for on in (False, True, False, True, True):
        buf.zero_()
        model.set_layer_timeline(buf if on else None)
        kv.set_len([40])
        out = sd.spec_step(model, kv, tree, words, out=out)
        torch.cuda.synchronize()
        assert bool(buf.any()) == on
    model.set_layer_timeline(None)
    model.set_graph_mode(False)
    assert kv.len() == [40 + int(out.n_accept[0])]
