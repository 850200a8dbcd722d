"""The decode runner works on its present state: a state attribute bound to
another tensor takes effect at the next call, after any number of earlier ones,
for every call that reads or writes it.  The library's calls are recorded, not
made (no GPU)."""

import dataclasses

import pytest
import torch

from paper_2602_08329_amd import binding as B
from paper_2602_08329_amd import schedule, synth

STATE = ["topk_idx", "topk_len", "anchor_set", "anchor_len", "shared_set", "shared_len"]


def used(runner, j):
    """Data pointers that one whole step hands to the library."""
    runner.step(j)
    ptrs = {a.data_ptr() for a in runner.seen if isinstance(a, torch.Tensor)}
    runner.seen.clear()
    return ptrs


@pytest.fixture
def runner(monkeypatch):
    inp = synth.random_inputs(2, 4, 2, 64, (90, 70), steps=3, seed=3)
    inp.w = dataclasses.replace(inp.w, k=8, window=4, sink=2, s=4)
    r = schedule.DecodeRunner(inp, device="cpu")
    r.seen = []
    for name in ("prhs_select", "prhs_select_shared", "prhs_dilate_reuse",
                 "prhs_sparse_decode_attn", "prhs_reuse_decode_attn"):
        monkeypatch.setattr(B, name, lambda *a, **k: r.seen.extend(a))
    return r


@pytest.mark.parametrize("per_step", [False, True])
@pytest.mark.parametrize("name", STATE + ["seq_lens"])
def test_state_bound_anew_is_used(runner, name, per_step):
    runner.per_step_sets = per_step
    used(runner, 0), used(runner, 1)
    old = getattr(runner, name)
    setattr(runner, name, old.clone())
    new = getattr(runner, name)

    def rows(t):
        return {x.data_ptr() for x in t}
    seen = used(runner, 0) | used(runner, 1)
    if name == "seq_lens":   # read as the anchor's lengths (the caches keep their own)
        assert new[0].data_ptr() in seen
    else:
        assert rows(new) <= seen
    assert not rows(old) & seen


def test_in_place_writes_show(runner):
    used(runner, 0)
    runner.anchor_len.fill_(7)
    assert bool((runner.set_for(0, 0)[1] == 7).all())
