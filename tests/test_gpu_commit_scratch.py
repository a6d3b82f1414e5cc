"""sd_kv_commit_rows at the edges of what the last pass left: sequences that were not part of it, and slots at or past a
sequence's own rows. Pure copies, so everything is bit-exact."""
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


def _model(sd, dtype):
    shape = dataclasses.replace(wl.preset("tiny").model, dtype=dtype)
    return shape, sd.Model(shape, {k: v.cuda() for k, v in wl.make_weights(shape).items()}, 256)


def _i32(x):
    return torch.tensor(x, dtype=torch.int32, device="cuda")


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_a_sequence_that_the_last_pass_did_not_hold_commits_nothing(sd, dtype):
    """Ragged prompts whose last pass holds one sequence: asked for two rows of each, only that one grows."""
    shape, model = _model(sd, dtype)
    lens, cap = [3, 300, 17], 330
    kv = sd.KVCache(model, 3, cap)
    sd.prefill(model, kv, torch.from_numpy(wl.zipf_prompt(shape.vocab, sum(lens))).cuda(), lens)
    past = [[t.clone() for t in kv.read_rows(shape.n_layers - 1, b, lens[b], 8)] for b in range(3)]
    sd.kv_commit_rows(model, kv, _i32([[0, 1]] * 3), _i32([2, 2, 2]))
    assert kv.len() == [3, 302, 17]
    for b in (0, 2):
        assert all(torch.equal(x, y) for x, y in zip(past[b], kv.read_rows(shape.n_layers - 1, b, lens[b], 8)))
    k, v = kv.read_rows(shape.n_layers - 1, 1, 300, 2)
    assert not torch.equal(k[0], k[1]) and bool(k.any())
    # the room that is asked for is judged for the whole batch, as it always was
    kv.set_len([3, 300, cap - 1])
    with pytest.raises(sd.SpecDecError) as e:
        sd.kv_commit_rows(model, kv, _i32([[0, 1]] * 3), _i32([2, 2, 0]))
    assert e.value.name == "SD_ERR_KV_FULL" and kv.len() == [3, 300, cap - 1]


def _slots_give_the_last_row(sd, dtype, fused, slots):
    shape, model = _model(sd, dtype)
    model.set_fused(fused)
    B, T, lens = 3, 5, [40, 7, 64]
    kv = sd.KVCache(model, B, 100)
    sd.prefill(model, kv, torch.from_numpy(wl.zipf_prompt(shape.vocab, sum(lens))).cuda(), lens)
    tree = sd.Tree(*wl.default_tree(T, shape.n_medusa, shape.topk), shape.n_medusa, shape.topk)
    words = torch.zeros((shape.vocab + 31) // 32, dtype=torch.int32, device="cuda")
    g = np.random.default_rng(8)
    kv.set_draft(g.integers(shape.vocab, size=B), g.integers(shape.vocab, size=(B, shape.n_medusa, shape.topk)))
    sd.spec_step(model, kv, tree, words)
    _check(sd, shape, model, kv, lens, T - 1, slots)
    # a prompt pass that holds the sequences' 3, 1 and 4 rows
    kv.set_len(lens)
    sd.prefill(model, kv, torch.from_numpy(wl.zipf_prompt(shape.vocab, 8)).cuda(), [3, 1, 4])
    _check(sd, shape, model, kv, lens, [2, 0, 3], slots)


def _check(sd, shape, model, kv, lens, last, slots):
    B = len(lens)
    last = [last] * B if isinstance(last, int) else last
    kv.set_len(lens)
    sd.kv_commit_rows(model, kv, _i32([[x] for x in last]), _i32([1] * B))
    want = [[kv.read_rows(layer, b, lens[b], 1) for layer in range(shape.n_layers)] for b in range(B)]
    kv.set_len(lens)
    sd.kv_commit_rows(model, kv, _i32([slots] * B), _i32([len(slots)] * B))
    for b in range(B):
        for layer in range(shape.n_layers):
            for got, w in zip(kv.read_rows(layer, b, lens[b], len(slots)), want[b][layer]):
                for j in range(len(slots)):
                    assert torch.equal(got[j], w[0]), f"sequence {b}, layer {layer}: slot {slots[j]} is not row {last[b]}"


@pytest.mark.parametrize("dtype,fused", [("bf16", False), ("bf16", True), ("f32", False)])
def test_slots_past_a_sequences_rows_give_its_last_row(sd, dtype, fused):
    _slots_give_the_last_row(sd, dtype, fused, [5, 31, 6])


@pytest.mark.parametrize("dtype,fused", [("bf16", False), ("bf16", True), ("f32", False)])
def test_slots_past_the_scratch_give_the_last_row_too(sd, dtype, fused):
    _slots_give_the_last_row(sd, dtype, fused, [32, 256, 2 ** 31 - 1])
