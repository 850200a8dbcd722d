"""The binding's native marshalling (_prhs_host) against its Python path: the
same outputs from both, the same exceptions for arguments that do not fit,
and the Python path for arguments the native one leaves to it."""

import math

import pytest
import torch

from paper_2602_08329_amd import binding as B
from paper_2602_08329_amd import synth

pytestmark = pytest.mark.gpu
DEV = "cuda"


@pytest.fixture(scope="module", autouse=True)
def gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    B.lib()


def case(dtype="bf16"):
    lens = (300, 77)
    inp = synth.random_inputs(2, 8, 2, 64, lens, dtype=dtype, paged=dtype == "bf16", seed=5,
                              device=DEV)
    n = torch.tensor(lens, dtype=torch.int32, device=DEV)
    return inp, B.KV(inp.K[0], inp.V[0], n, inp.w.capacity, 8, inp.block_table), n


def run_all(inp, kv, n):
    """Outputs of one call of every entry point that takes the extension."""
    q, scale = inp.q[0, 0], 1 / math.sqrt(64)
    p = B.params(k=30, sink=4, window=8, refresh_every=4)
    i32 = dict(dtype=torch.int32, device=DEV)
    kc, sc = B.prhs_max_topk(p, inp.w.capacity), B.prhs_set_capacity(p, inp.w.capacity)
    ws = B.workspace(B.prhs_workspace_size(B.PRHS_OP_SELECT, kv, p), DEV)
    wa = B.workspace(max(B.prhs_workspace_size(B.PRHS_OP_SPARSE_ATTN, kv, p, sc),
                         B.prhs_workspace_size(B.PRHS_OP_DENSE_ATTN, kv)), DEV)
    res = []

    def keep(*shape, dtype=torch.int32):
        res.append(torch.zeros(*shape, dtype=dtype, device=DEV))
        return res[-1]

    def out():
        return keep(2, 8, 64, dtype=torch.float32), keep(2, 8, dtype=torch.float32)

    sel = lambda: (keep(2, 2, kc), keep(2, 2), keep(2, 2, sc), keep(2, 2))  # noqa: E731
    B.prhs_select(kv, q, p, *sel(), ws)
    top, tl, st, sl = sel()
    sh, hl = keep(2, 2, sc), keep(2, 2)
    B.prhs_select_shared(kv, q, p, top, tl, st, sl, sh, hl, ws)
    flat = lambda v: torch.full((4,), v, **i32)  # noqa: E731
    B.prhs_select_gated(kv, q, p, flat(-1), *sel(), keep(2, 2, sc), keep(2, 2), ws)
    B.prhs_gate_select(kv, q, p, 0.8, 0, torch.zeros(3, 2, 8, 64, dtype=q.dtype, device=DEV),
                       keep(3, 4), keep(3, 2), keep(4), keep(4), keep(4), keep(4), *sel(),
                       keep(2, 2, sc), keep(2, 2), ws)
    B.prhs_dilate_reuse(p, top, tl, n, n, keep(2, 2, sc), keep(2, 2))
    B.prhs_sparse_decode_attn(kv, q, st, sl, scale, *out(), wa)
    B.prhs_sparse_decode_attn_static(kv, q, st, sl, scale, *out())
    B.prhs_reuse_decode_attn(kv, q, sh, hl, n, scale, *out(), wa)
    B.prhs_dense_decode_attn(kv, q, scale, out()[0], None, wa)
    ps = B.psaw(3, 4, 1, 0.5, 1.0, 4)
    ids, tail = torch.arange(4, **i32), n.repeat_interleave(2).contiguous()
    B.prhs_pool_decode_attn(kv, q, sh, hl, ids, tail, scale, *out(), wa, psaw=ps)
    B.prhs_pool_decode_attn(kv, q, sh, hl, ids, tail, scale, *out(), wa, unit_gate=flat(1),
                            units_side=B.PRHS_UNITS_SHARING)
    if q.dtype == torch.bfloat16:
        qq = q[:, :, None].expand(2, 8, 9, 64).contiguous()
        B.prhs_prefill_attn(kv, qq, scale, keep(2, 8, 9, 64, dtype=torch.float32),
                            keep(2, 8, 9, dtype=torch.float32), psaw=ps)
    torch.cuda.synchronize()
    return res


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_native_marshalling_equals_python(dtype, monkeypatch):
    c = case(dtype)
    host, taken = B._host, []

    class Watch:
        def __getattr__(self, name):
            def f(*a):
                r = getattr(host, name)(*a)
                if r is not None:
                    taken.append(name)
                return r
            return f

    monkeypatch.setattr(B, "_host", Watch())
    native = run_all(*c)
    names = {"select", "select_shared", "select_gated", "gate_select", "dilate_reuse", "sparse",
             "reuse", "dense", "pool"} | ({"prefill"} if dtype == "bf16" else set())
    assert set(taken) == names
    monkeypatch.setattr(B, "_host", None)
    for x, y in zip(native, run_all(*c)):
        assert torch.equal(x, y)


def test_what_does_not_fit_raises_as_before():
    inp, kv, n = case()
    q, scale = inp.q[0, 0], 0.125
    st = torch.zeros(2, 2, 40, dtype=torch.int32, device=DEV)
    sl = torch.full((2, 2), 20, dtype=torch.int32, device=DEV)
    out = torch.zeros(2, 8, 64, device=DEV)
    wa = B.workspace(B.prhs_workspace_size(B.PRHS_OP_SPARSE_ATTN, kv, None, 40), DEV)
    call = lambda q=q, st=st, sl=sl, scale=scale, out=out, wa=wa: B.prhs_sparse_decode_attn(  # noqa: E731
        kv, q, st, sl, scale, out, None, wa)
    call()
    for bad in (dict(q=q.float()), dict(q=q[:, :4]), dict(st=st.long()), dict(sl=sl[0]),
                dict(st=st.transpose(0, 1)), dict(out=out.cpu()), dict(wa=wa[None])):
        with pytest.raises(ValueError):
            call(**bad)
    with pytest.raises(TypeError):
        call(q=None)
    with pytest.raises(B.PrhsError):
        call(wa=wa[:0])
    with pytest.raises(B.PrhsError):
        call(scale=float("nan"))
    # arguments the Python path takes: a tensor subclass, a whole number
    ref = out.clone()
    call(q=torch.nn.Parameter(q, requires_grad=False))
    assert torch.equal(out, ref)
    call(scale=torch.tensor(0.125))
    assert torch.equal(out, ref)
