"""sd_kv_commit_rows at the edges of what the last pass left: sequences that were not part of it.
Pure copies, so everything is bit-exact."""
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
