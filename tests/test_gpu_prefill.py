"""GPU parity of prefill attention under the PSAW mask (prhs_prefill_attn)
against the oracle's prefill_attention: plain causal layers and pruning
layers, GQA and MHA, d 64 and 128, ragged prompts (rows past a prompt are
empty), query spans shorter than the prompt, contiguous and paged caches,
and sampled rows of a full
LLaMA-2-7B-shaped 4k prefill and of launches large enough to take the
256-query blocks.  Outputs within 2e-3 of the fp64 oracle per
(batch, head, query) row in the max norm, lse within 1e-4."""

import math

import numpy as np
import pytest
import torch

import oracle as O
from paper_2602_08329_amd import binding as B
from paper_2602_08329_amd import synth
from tests.test_prefill_plan import FORMS, WINDOW

pytestmark = pytest.mark.gpu
DEV = "cuda"
TOL = 2e-3


@pytest.fixture(scope="module", autouse=True)
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    B.lib()


def _queries(batch, hq, T, d, seed):
    gen = torch.Generator(device="cpu")
    gen.manual_seed(seed)
    return synth._round_grid(torch.randn(batch, hq, T, d, generator=gen)).to(torch.bfloat16)


def run_prefill(batch, hq, hkv, d, lens, T, psaw=None, layer=None, n_layers=None, sink=4,
                seed=0, rows=None, heads=None, paged=False, page_size=16):
    """psaw = (l_s, phi, alpha) with layer / n_layers: the layer's window of
    Eq. psaw, which the library evaluates; the oracle's first visible
    positions are the reference."""
    inp = synth.random_inputs(batch, hq, hkv, d, lens, seed=seed, device=DEV, paged=paged,
                              page_size=page_size)
    cap = inp.w.capacity
    seq = torch.tensor(lens, dtype=torch.int32, device=DEV)
    kv = B.KV(inp.K[0], inp.V[0], seq, cap, hq, inp.block_table)
    q = _queries(batch, hq, T, d, seed + 1).to(DEV)
    ps = None if psaw is None else B.psaw(layer, n_layers, *psaw, sink)
    out = torch.full((batch, hq, T, d), float("nan"), device=DEV)
    lse = torch.full((batch, hq, T), float("nan"), device=DEV)
    scale = 1.0 / math.sqrt(d)
    B.prhs_prefill_attn(kv, q, scale, out, lse, psaw=ps)
    torch.cuda.synchronize()
    y, ls = out.cpu().numpy(), lse.cpu().numpy()
    qh = q.float().cpu().numpy()
    vis_h = None
    if psaw is not None:
        vis_h = O.psaw_prefill_visible(layer, n_layers, T, sink, *psaw)
    else:
        sink = 0
    G = hq // hkv
    worst = 0.0
    for b in range(batch):
        n = min(lens[b], T)
        units = {g: synth.gather_unit(inp, 0, b, g, max(n, 1)) for g in range(hkv)}
        for h in (range(hq) if heads is None else heads):
            g = h // G
            Kg, Vg = units[g]
            if rows is None:
                yr, lr = O.prefill_attention(qh[b, h], Kg, Vg, n, sink=sink,
                                             vis_start=vis_h, scale=scale)
                check_rows = range(T)
            else:
                check_rows = [i for i in rows if i < T]
                yr = np.zeros((T, d))
                lr = np.full(T, -np.inf)
                for i in check_rows:
                    if i < n:
                        S = O.prefill_visible_set(i, sink, None if vis_h is None else int(vis_h[i]))
                        yr[i], lr[i] = O.sparse_attention(qh[b, h, i], Kg[: i + 1],
                                                          Vg[: i + 1], S, scale)
            for i in check_rows:
                if i >= n:
                    assert np.all(y[b, h, i] == 0) and ls[b, h, i] == -np.inf, (b, h, i)
                    continue
                den = max(np.abs(yr[i]).max(), 1e-30)
                e = np.abs(y[b, h, i] - yr[i]).max() / den
                worst = max(worst, e)
                assert e <= TOL, f"b{b} h{h} row {i}: rel err {e:.3e}"
                assert ls[b, h, i] == lr[i] or abs(ls[b, h, i] - lr[i]) <= 1e-4 * max(1.0, abs(lr[i])), \
                    (b, h, i)
    print(f"prefill worst relative error {worst:.2e}")
    return worst


def test_prefill_causal_mha_ragged():
    # plain causal attention; the second prompt ends inside a query block
    run_prefill(2, 4, 4, 128, (300, 129), 300)


def test_prefill_psaw_top_layer_gqa():
    # top layer of 8 with a strong window (phi 0.3): most early keys masked
    run_prefill(2, 8, 2, 128, (777, 640), 777, psaw=(6, 0.3, 1.0), layer=7, n_layers=8, sink=4,
                seed=3)


def test_prefill_psaw_mid_layer_d64():
    run_prefill(1, 4, 4, 64, (500,), 500, psaw=(4, 0.5, 1.5), layer=5, n_layers=8, sink=2, seed=5)


def test_prefill_below_pruning_depth_is_causal():
    # a layer below l_s: vis_start is the sink end everywhere
    run_prefill(1, 4, 2, 128, (260,), 260, psaw=(6, 0.7, 1.0), layer=2, n_layers=8, sink=4, seed=7)


def test_prefill_query_span_shorter_than_prompt():
    # q covers positions [0, 150) of prompts of 400 and 90 tokens
    run_prefill(2, 4, 4, 128, (400, 90), 150, psaw=(2, 0.4, 1.0), layer=3, n_layers=4, sink=4,
                seed=9)


@pytest.mark.parametrize("T,sink", [(1, 4), (64, 0), (65, 1), (33, 40), (192, 3), (193, 70)])
def test_prefill_small_and_block_edges(T, sink):
    run_prefill(1, 2, 1, 128, (T,), T, psaw=(1, 0.2, 1.0), layer=1, n_layers=2, sink=sink,
                seed=11 + T)


def test_prefill_full_size_llama2_4k_sampled():
    # LLaMA-2-7B shape (32 heads, d 128), one 4k prompt, the top layer with
    # the Sec. 5.1 defaults; sampled rows of a few heads against the oracle
    T = 4096
    rows = [0, 1, 63, 64, 1000, 2047, 3000, 4031, 4095]
    run_prefill(1, 32, 32, 128, (T,), T, psaw=(24, 0.7, 1.0), layer=31, n_layers=32, sink=4,
                seed=13, rows=rows, heads=[0, 17, 31])


@pytest.mark.parametrize("d", [128, 64])
def test_prefill_wide_blocks_sampled(d):
    # enough (batch, head) units that the launch takes 256-query blocks
    # (at least 4 workgroups per CU); ragged prompts, GQA, a pruning layer
    lens = (1024, 1000, 777, 1024, 600, 1024, 513, 1024)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    assert -(-1024 // 256) * len(lens) * 32 >= 4 * cus
    rows = [0, 1, 255, 256, 511, 512, 776, 777, 999, 1023]
    run_prefill(8, 32, 8, d, lens, 1024, psaw=(6, 0.5, 1.0), layer=7, n_layers=8, sink=16,
                seed=17 + d, rows=rows, heads=[0, 13, 31])


def test_prefill_paged_psaw_gqa():
    # a paged cache (16-token pages in a seeded random order), ragged prompts
    run_prefill(2, 8, 2, 128, (777, 300), 777, psaw=(6, 0.3, 1.0), layer=7, n_layers=8, sink=4,
                seed=21, paged=True)


def test_prefill_paged_causal_d64_small_pages():
    run_prefill(3, 4, 4, 64, (129, 64, 250), 250, sink=2, seed=23, paged=True, page_size=8)


def test_prefill_paged_wide_blocks_sampled():
    lens = (1024, 1000, 777, 1024, 600, 1024, 513, 1024)
    rows = [0, 255, 256, 599, 776, 1023]
    run_prefill(8, 32, 8, 128, lens, 1024, psaw=(6, 0.5, 1.0), layer=7, n_layers=8, sink=16,
                seed=25, rows=rows, heads=[0, 31], paged=True)


@pytest.mark.parametrize("sink,phi,alpha", [(0, 0.01, 3.0), (5, 0.01, 3.0), (3, 0.9, 0.05),
                                             (70, 0.2, 1.0)])
def test_prefill_extreme_windows(sink, phi, alpha):
    # windows far from the defaults: phi^alpha = 1e-6 leaves each row its sink
    # and the two keys [i - 1, i] (first visible position i - 1 at the top
    # layer), a small exponent masks almost nothing, a sink wider than early
    # rows; ragged prompts and block edges
    T = 450
    run_prefill(2, 4, 2, 128, (450, 333), T, psaw=(2, phi, alpha), layer=3, n_layers=4, sink=sink,
                seed=33)


def test_prefill_rejects_fp32():
    inp = synth.random_inputs(1, 2, 2, 64, (40,), dtype="f32", seed=1, device=DEV)
    seq = torch.tensor((40,), dtype=torch.int32, device=DEV)
    kv = B.KV(inp.K[0], inp.V[0], seq, inp.K[0].shape[2], 2)
    q = torch.zeros(1, 2, 40, 64, device=DEV)
    out = torch.zeros(1, 2, 40, 64, device=DEV)
    with pytest.raises(B.PrhsError) as e:
        B.prhs_prefill_attn(kv, q, 0.125, out)
    assert e.value.status == B.PRHS_E_UNSUPPORTED


@pytest.mark.parametrize("batch,hq,T,d,paged", [
    (1, 2, 127, 128, False),    # one block of 128 queries, 16 a wave, two 64-key tiles
    (1, 2, 129, 64, True),      # 16-query waves, two blocks of 80
    (3, 24, 257, 128, True),    # two key sides: 128-query blocks (on 256 CUs)
    (3, 24, 384, 64, False),
    (3, 60, 255, 128, False),   # one key side: 256-query blocks, units not a multiple of the XCDs
    (5, 24, 321, 128, True),    # units a multiple of the XCDs
    (2, 64, 537, 128, False),   # a first block smaller than the others
    (1, 60, 97, 64, True),      # blocks smaller than their waves allow
    (2, 64, 173, 128, True),    # 16-query waves, two blocks
    (2, 64, 265, 64, False),
    (1, 64, 113, 128, False),   # 16-query waves, one block with a wave to spare
    (4, 64, 300, 64, False),    # d 64, two workgroups a CU: one key side
    (1, 48, 300, 64, True),     # and four
])
def test_prefill_key_sides_and_block_order(batch, hq, T, d, paged):
    # outputs as for every other prefill test: bf16 hi + lo probabilities
    lens = tuple(max(1, T - 61 * i) for i in range(batch))
    rows = sorted({0, 31, 32, 63, 64, 127, 128, 191, 192, 255, 256, T // 2, T - 62, T - 1})
    run_prefill(batch, hq, min(hq, 4), d, lens, T, psaw=(2, 0.6, 1.0), layer=3, n_layers=4, sink=5,
                seed=41 + T, rows=[r for r in rows if 0 <= r < T], heads=[0, hq // 2, hq - 1],
                paged=paged)


@pytest.mark.parametrize("w,ns,d,paged,batch,hq,T", FORMS)
def test_prefill_every_form(w, ns, d, paged, batch, hq, T):
    # rows at the edges of 32- and 64-query waves, of blocks and of 128-key tiles
    lens = tuple(max(1, T - 61 * i) for i in range(batch))
    rows = sorted({r for e in range(0, T + 1, 64) for r in (e - 1, e)} | {16, 31, 32, 33, T // 2, T - 62, T - 1})
    rows = [r for r in rows if 0 <= r < T] if T < 900 else [0, 31, 255, 256, 511, 512, 767, 768, 939, T - 1]
    run_prefill(batch, hq, min(hq, 4), d, lens, T, seed=51 + T, rows=rows, heads=[0, hq // 2, hq - 1],
                paged=paged, **WINDOW)


def test_prefill_order_in_several_groups():
    # 40 units an XCD in groups of 20, the last block of each prompt short; and 5 an
    # XCD, fewer blocks than its CUs
    for batch, hq, T in ((4, 80, 1790), (1, 40, 600)):
        run_prefill(batch, hq, 8, 64, (T,) * batch, T, seed=61 + T, rows=[0, 255, 256, T - 255, T - 1],
                    heads=[0, 1, hq // 2, hq - 1])
