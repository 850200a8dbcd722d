"""Decode attention around the lines of its split rules, against the oracle:
launches of many units, unsplit, in a few splits, and a few units more than the
CUs, with lengths at the edges of what a workgroup takes.  Which splits a launch
takes is checked beside it, so that a rule that moves does not leave a form
untested."""

import numpy as np
import pytest
import torch

import oracle as O
from paper_2602_08329_amd import binding as B
from paper_2602_08329_amd import synth
from tests.test_attention_splits import CUS, f32_heads, splits
from tests.test_gpu_parity import TOL, assert_close, run_dense, run_sparse

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.fixture(scope="module", autouse=True)
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    B.lib()


def check_dense(inp, lens, y, lse, dtype, some):
    g = inp.w.hq // inp.w.hkv
    for b, hk in some:
        K, V = synth.gather_unit(inp, 0, b, hk, lens[b])
        Qg = synth.query_group(inp, 0, 0, b, hk)
        for j in range(g):
            h = hk * g + j
            yr, lr = O.dense_attention(Qg[j], K, V)
            assert_close(y[b, h], lse[b, h], yr, lr, TOL[dtype], f"dense b{b} h{h} n{lens[b]}")


@pytest.mark.parametrize("batch,hq,hkv,d,paged,n,want", [
    (129, 1, 1, 64, False, 2048, 1),     # unsplit: all rows a workgroup stages
    (200, 2, 1, 64, True, 2049, 6),      # one more: split
    (136, 1, 1, 64, False, 2500, 7),     # not eight, a few over twice 512 workgroups
    (257, 1, 1, 64, False, 1279, 1),     # a few more units than CUs: short units unsplit,
    (257, 1, 1, 64, True, 1280, 4),      # longer ones split
    (65, 10, 5, 64, False, 700, 1),      # 325 units
])
def test_dense_many_units(batch, hq, hkv, d, paged, n, want):
    # lengths from 1 to n, some at the edges of the last split
    lens = tuple([n, 1, n - 1, 32, n // want, min(n, n // want + 1)][b] if b < 6 else max(1, n - 37 * b)
                 for b in range(batch))
    inp = synth.random_inputs(batch, hq, hkv, d, lens, paged=paged, page_size=16, seed=701 + n, device=DEV)
    assert splits("bf16", batch, hq, hkv, d, inp.w.capacity, True) == want
    y, lse = run_dense(inp, lens)
    assert not np.isnan(y).any()
    check_dense(inp, lens, y, lse, "bf16", [(b, b % hkv) for b in (*range(6), batch // 2, batch - 1)])


F32_FORMS = [
    # heads a workgroup of sets and of the stream, batch, hq, hkv, d, paged, rows: every
    # head count of the fp32 kernel, whole, short of it (3, 5, 9 heads) and in several
    # workgroups a unit
    (1, 1, 1, 8, 1, 128, False, 377),
    (2, 2, 4, 32, 4, 64, True, 90),
    (4, 4, 16, 64, 16, 64, False, 300),
    (4, 4, 16, 48, 16, 128, True, 260),
    (4, 4, 16, 64, 4, 128, False, 100),
    (8, 8, 24, 64, 4, 128, False, 100),
    (8, 8, 16, 80, 16, 128, False, 270),
    (8, 8, 4, 128, 8, 64, False, 1100),
    (8, 8, 16, 144, 16, 64, True, 300),
    (8, 8, 17, 64, 8, 64, True, 1200),   # the stream unsplit
]


@pytest.mark.parametrize("sets_gp,dense_gp,batch,hq,hkv,d,paged,rows", F32_FORMS)
def test_f32_heads_per_workgroup(sets_gp, dense_gp, batch, hq, hkv, d, paged, rows):
    if torch.cuda.get_device_properties(0).multi_processor_count == CUS:
        assert f32_heads(batch, hq, hkv, d, rows, False) == sets_gp
        assert f32_heads(batch, hq, hkv, d, rows, True) == dense_gp
    lens = tuple(max(1, rows - (b * 41) % rows) for b in range(batch))
    inp = synth.random_inputs(batch, hq, hkv, d, lens, dtype="f32", paged=paged, page_size=8,
                              seed=801 + rows, device=DEV)
    assert inp.w.capacity == rows
    rng = np.random.default_rng(rows)
    sets = {(b, g): sorted(rng.choice(n, size=int(rng.integers(1, n + 1)) if b else n, replace=False).tolist())
            for b, n in enumerate(lens) for g in range(hkv)}
    y, lse = run_dense(inp, lens)
    z, zse = run_sparse(inp, lens, sets, rows)
    assert not np.isnan(y).any() and not np.isnan(z).any()
    some = [(0, 0), (0, hkv - 1), (batch // 2, hkv // 2), (batch - 1, hkv - 1)]
    check_dense(inp, lens, y, lse, "f32", some)
    g = hq // hkv
    for b, hk in some:
        K, V = synth.gather_unit(inp, 0, b, hk, lens[b])
        Qg = synth.query_group(inp, 0, 0, b, hk)
        for j in range(g):
            h = hk * g + j
            yr, lr = O.sparse_attention(Qg[j], K, V, sets[(b, hk)])
            assert_close(z[b, h], zse[b, h], yr, lr, TOL["f32"], f"sparse b{b} h{h}")
