"""Lengths and drafts are set in stream order without the host waiting: what the caller passed may go away at once."""
import dataclasses

import numpy as np
import pytest
import torch

import workload as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_inputs_may_go_away_at_once(dtype):
    """On a side stream that is busy, from tensors of the default stream: deleted after the call, their memory offered to the
    default stream and overwritten there; lengths from a list that is changed afterwards. The last setting counts."""
    import paper_2503_14153_amd as sd
    shape = dataclasses.replace(wl.preset("tiny").model, dtype=dtype)
    model = sd.Model(shape, {k: v.cuda() for k, v in wl.make_weights(shape).items()}, 64)
    B = 3
    kv = sd.KVCache(model, B, 100)
    g = np.random.default_rng(3)
    side, busy = torch.cuda.Stream(), torch.randn(4096, 4096, device="cuda")
    for _ in range(3):
        root = torch.from_numpy(g.integers(shape.vocab, size=B).astype(np.int32)).cuda()
        cand = torch.from_numpy(g.integers(shape.vocab, size=(B, shape.n_medusa, shape.topk)).astype(np.int32)).cuda()
        want = root.cpu(), cand.cpu()
        lens = [1, 2, 3]
        torch.cuda.synchronize()
        with torch.cuda.stream(side):
            for _ in range(4):
                busy @ busy
            kv.set_len([9, 9, 9])
            kv.set_len(lens)
            kv.set_draft(root, cand)
        lens[:] = [50, 50, 50]
        sizes = root.shape, cand.shape
        del root, cand
        junk = [torch.full(s, -7, dtype=torch.int32, device="cuda") for s in sizes for _ in range(8)]
        with torch.cuda.stream(side):
            got = kv.get_draft()
            assert kv.len() == [1, 2, 3]
        assert all(torch.equal(a.cpu(), b) for a, b in zip(got, want))
        del junk


def test_refused_under_capture():
    """A replay would set what the host has other bounds on, or read temporaries that are gone; the capture itself goes on."""
    import paper_2503_14153_amd as sd
    shape = wl.preset("tiny").model
    model = sd.Model(shape, {k: v.cuda() for k, v in wl.make_weights(shape).items()}, 64)
    kv = sd.KVCache(model, 1, 100)
    kv.set_len([7])
    root = torch.zeros(1, dtype=torch.int32, device="cuda")
    cand = torch.zeros(1, shape.n_medusa, shape.topk, dtype=torch.int32, device="cuda")
    x, graph = torch.zeros(4, device="cuda"), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        x += 1
        with pytest.raises(Exception, match="captured"):
            kv.set_len([9])
        with pytest.raises(RuntimeError, match="captured"):
            kv.set_draft(root, cand)
    for n in (1, 2):
        graph.replay()
        torch.cuda.synchronize()
        assert x.tolist() == [float(n)] * 4
    assert kv.len() == [7]
