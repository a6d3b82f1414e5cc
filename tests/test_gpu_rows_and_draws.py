"""Cache rows in natural layout at every alignment, and inverse-CDF draws around the sizes where their kernels change."""
import dataclasses

import numpy as np
import pytest
import torch

import workload as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("name", ["tiny", "7b"])           # head_dim 64, 128
@pytest.mark.parametrize("offset", [0, 1, 4])              # elements the caller's arrays are off 16-byte alignment by
def test_rows_of_any_range_and_alignment(name, offset):
    """Ranges that start and end anywhere in a 32-row block and in an eight-row value piece: what was written is read back,
    bit for bit, and no other row of the cache changes."""
    import paper_2503_14153_amd as sd
    shape = dataclasses.replace(wl.preset("tiny").model, dtype="bf16", n_layers=1, n_heads=3,
                                head_dim=wl.preset(name).model.head_dim, d_model=3 * wl.preset(name).model.head_dim, d_ffn=64)
    model = sd.Model(shape, {k: v.cuda() for k, v in wl.make_weights(shape).items()}, 32)
    cap = 150
    kv = sd.KVCache(model, 2, cap)
    g = torch.Generator(device="cuda").manual_seed(9)

    def rows(n):
        flat = torch.randn(n * 3 * shape.head_dim + 8, generator=g, device="cuda").bfloat16()
        return flat[offset: offset + n * 3 * shape.head_dim].view(n, 3, shape.head_dim)

    want = [torch.zeros((cap, 3, shape.head_dim), dtype=torch.bfloat16, device="cuda") for _ in range(2)]
    for row0, n in [(0, cap), (0, 1), (31, 2), (5, 27), (32, 32), (33, 62), (4, 4), (12, 8), (149, 1), (90, 41), (17, 15)]:
        k, v = rows(n), rows(n)
        assert (k.data_ptr() % 16 == 0) == (offset == 0)
        kv.write_rows(0, 1, row0, k, v)
        want[0][row0: row0 + n], want[1][row0: row0 + n] = k, v
        for a, m in [(0, cap), (row0, n), (max(row0 - 3, 0), 1)]:
            out = [rows(m), rows(m)]                       # read into arrays of the same alignment
            sd.binding._check(sd.lib().sd_kv_read_rows(kv.handle, 0, 1, a, m, out[0].data_ptr(), out[1].data_ptr(),
                                                       torch.cuda.current_stream().cuda_stream))
            for got, w in zip(out, want):
                assert torch.equal(got, w[a: a + m])
    assert float(kv.read_rows(0, 0, 0, cap)[0].abs().max()) == 0.0      # the other sequence


@pytest.mark.parametrize("vocab", [1, 63, 64, 65, 1000, 4096, 4097, 16385, 32016, 32769, 65537, 163840])
def test_draws_fall_into_their_interval(vocab):
    """The id drawn at u is the one whose interval of the cumulative distribution (float64) holds u; ends of the range and
    of the ids included, and rows with ids that have no mass. Bound: the weights are float32 (2^-24 each, and as much
    again from the exponential's argument times |x| <= 88), so boundaries move by less than 2e-5."""
    import paper_2503_14153_amd as sd
    g = torch.Generator(device="cuda").manual_seed(vocab)
    logits = torch.randn((3, vocab), generator=g, device="cuda") * 3
    if vocab > 2:
        logits[1, : vocab // 2] = -float("inf")
        logits[2, 1:] = -200.0                             # all mass on id 0
    us = torch.tensor([0.0, 1e-7, 0.25, 0.5, 0.75, 0.999999, 1 - 2 ** -24], device="cuda")
    rows = torch.arange(3, device="cuda", dtype=torch.int32).repeat_interleave(len(us))
    got = sd.sample_tokens(logits, rows, us.repeat(3), 0.8).cpu().numpy()
    p = torch.softmax(logits.double() / 0.8, -1).cpu().numpy()
    F = np.cumsum(p, -1)
    for i, t in enumerate(got):
        r, u = i // len(us), float(us[i % len(us)])
        assert 0 <= t < vocab and p[r, t] > 0
        assert (F[r, t - 1] if t else 0.0) - 2e-5 <= u < F[r, t] + 2e-5


@pytest.mark.parametrize("vocab,stride", [(32016, 3 * 64), (32016, 67), (65537, 5 * 64), (163840, 1000)])
def test_draws_over_rows_that_are_mostly_masked(vocab, stride):
    """One id in `stride` has mass (groups of 64 ids without any in between): every draw is an id that has, and the one whose
    interval holds u (bound as above)."""
    import paper_2503_14153_amd as sd
    g = torch.Generator(device="cuda").manual_seed(stride)
    logits = torch.full((1, vocab), -float("inf"), device="cuda")
    logits[0, 7::stride] = torch.randn(len(range(7, vocab, stride)), generator=g, device="cuda") * 3
    us = torch.cat([torch.rand(2000, generator=g, device="cuda"), torch.tensor([0.0, 0.5, 1 - 2 ** -24], device="cuda")])
    rows = torch.zeros(len(us), device="cuda", dtype=torch.int32)
    got = sd.sample_tokens(logits, rows, us, 0.8).cpu().numpy()
    F = np.cumsum(torch.softmax(logits.double() / 0.8, -1).cpu().numpy()[0])
    u = us.cpu().numpy()
    assert (got >= 7).all() and (got < vocab).all() and ((got - 7) % stride == 0).all()
    assert (F[got - 1] - 2e-5 <= u).all() and (u < F[got] + 2e-5).all()
