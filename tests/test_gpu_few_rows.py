"""Steps of one or two rows, whose O and down projections build their operands themselves, against steps of more rows."""
import dataclasses

import numpy as np
import pytest
import torch

import workload as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,T", [(1, 1), (2, 1), (1, 2), (3, 1), (1, 5)])       # one and two rows; a few more
@pytest.mark.parametrize("width", ["7b", "13b", "hd64"])
def test_few_rows_match_the_same_sequences_among_more(B, T, width):
    """Reference: the same sequences with others beside them (eight sequences: the operand comes from memory). Row sums
    are taken in the same order on both sides, but attention splits its rows differently (float32 sums in another order,
    a flipped bfloat16 rounding of the step's own keys and values): bound 2e-3 relative."""
    import paper_2503_14153_amd as sd
    base = wl.preset("13b" if width == "13b" else "7b", 1).model
    shape = dataclasses.replace(base, vocab=1000, n_medusa=3)
    if width == "hd64":
        shape = dataclasses.replace(shape, n_heads=24, head_dim=64, d_model=1536, d_ffn=4096)
    model = sd.Model(shape, wl.make_weights(shape, device="cuda"), 256)
    more = 8
    lens = [200, 3, 64, 33, 500, 31, 95, 1]
    g = np.random.default_rng(8)
    root, cand = g.integers(shape.vocab, size=more), g.integers(shape.vocab, size=(more, 3, shape.topk))
    words = torch.zeros((shape.vocab + 31) // 32, dtype=torch.int32, device="cuda")
    tree = sd.Tree(*wl.default_tree(T, 3, shape.topk), 3, shape.topk)
    out = []
    for n_seq in (B, more):
        kv = sd.KVCache(model, n_seq, 520)
        for b in range(n_seq):
            k, v = (wl.synthetic_kv_rows(3, f"{t}{b}", (lens[b], shape.n_heads, shape.head_dim), "bf16", "cuda") for t in "kv")
            kv.write_rows(0, b, 0, k, v)
        kv.set_len(lens[:n_seq])
        kv.set_draft(root[:n_seq], cand[:n_seq])
        out.append(sd.spec_step(model, kv, tree, words, want_logits=True).logits[:B])
    assert torch.isfinite(out[0]).all()
    assert float((out[0] - out[1]).norm() / out[1].norm()) < 2e-3
