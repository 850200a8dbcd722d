"""The refresh on either side of the rule that chooses between one fused launch
and scoring spread over the chip (on 256 CUs: long rows of up to five eighths of
the CUs, up to seven eighths under the similarity gate), against the oracle, and
the gated form against its separate launches."""

import pytest
import torch

from paper_2602_08329_amd import binding as B
from paper_2602_08329_amd import synth
from tests.test_gpu_parity import check_select, check_select_shared, kv_for

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.fixture(scope="module", autouse=True)
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    B.lib()


@pytest.mark.parametrize("rows,hkv,longest,paged", [
    (129, 1, 4000, False), (129, 1, 3999, True), (160, 8, 4001, True), (161, 1, 4000, True)])
def test_long_rows_around_the_line(rows, hkv, longest, paged):
    lens = tuple(max(1, longest - 61 * b) if b % 7 else longest for b in range(rows // hkv))
    inp = synth.random_inputs(len(lens), 2 * hkv, hkv, 64, lens, paged=paged, page_size=16,
                              seed=901 + rows, grid=True, device=DEV)
    assert inp.w.capacity == longest
    p = B.params(k=90, sink=4, window=34, refresh_every=1)
    check_select(inp, lens, p)
    check_select_shared(inp, lens, p)


@pytest.mark.parametrize("batch,paged", [(28, True), (28, False), (29, True)])
def test_gated_long_rows_equal_separate_launches(batch, paged):
    hkv, longest = 8, 4100   # 224 rows: scored over the chip after the gate; 232: fused
    lens = tuple(longest - 1 - 53 * b for b in range(batch))
    inp = synth.random_inputs(batch, 2 * hkv, hkv, 64, lens, paged=paged, page_size=16, seed=911,
                              grid=True, steps=2, device=DEV)
    p = B.params(k=60, sink=4, window=8, refresh_every=2)
    kc, sc = B.prhs_max_topk(p, inp.w.capacity), B.prhs_set_capacity(p, inp.w.capacity)
    i32 = dict(dtype=torch.int32, device=DEV)
    U = batch * hkv

    def state():
        gate = [torch.zeros(2, batch, 2 * hkv, 64, dtype=torch.bfloat16, device=DEV), torch.zeros(2, U, **i32),
                torch.zeros(2, batch, **i32)] + [torch.zeros(U, **i32) for _ in range(4)]
        sets = [torch.full((batch, hkv, cap), -7, **i32) if cap else torch.zeros(batch, hkv, **i32)
                for cap in (kc, 0, sc, 0, sc, 0)]
        return gate, sets

    (g0, s0), (g1, s1) = state(), state()
    for j in range(2):
        kv, t = kv_for(inp, [x + j for x in lens])
        ws = B.workspace(B.prhs_workspace_size(B.PRHS_OP_SELECT, kv, p), DEV)
        q = inp.q[0, j].clone()
        if j == 1:
            q[::2] = inp.q[0, 0][::2]   # close to the first step's
        B.prhs_gate_select(kv, q, p, 0.8, j, *g0, *s0, ws)
        B.prhs_gate(q, t, 0.8, j, *g1, hkv)
        B.prhs_select_gated(kv, q, p, g1[3], *s1, ws)
        torch.cuda.synchronize()
        for x, y in zip(g0 + s0, g1 + s1):
            assert torch.equal(x, y)
    assert bool((g0[3] >= 0).any()) and bool((g0[3] < 0).any())
