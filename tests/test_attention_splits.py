"""How the decode attention launches divide their rows, read on the host from
the workspace a call asks for (its split-K partials): no device work."""

import ctypes
import math
import random
import re

import pytest

from paper_2602_08329_amd import binding as B

CUS = 256


def kv(dtype, batch, hq, hkv, d, rows):
    return B.PrhsKv(batch, hq, hkv, d, B.PRHS_BF16 if dtype == "bf16" else B.PRHS_F32,
                    B.PRHS_KV_CONTIGUOUS, rows, 0, 0, 0, 0x1000, 0x2000, None, 0x3000, rows)


def need(dtype, batch, hq, hkv, d, rows, dense):
    """Bytes of workspace the call needs, from its refusal of none."""
    L, c = B.lib(), kv(dtype, batch, hq, hkv, d, rows)
    if dense:
        st = L.prhs_dense_decode_attn(ctypes.byref(c), 0x10, 1.0, 0x20, None, None, 0, None)
    else:
        st = L.prhs_sparse_decode_attn(ctypes.byref(c), 0x10, 0x20, 0x30, rows, 1.0, 0x40, None, None,
                                       0, None)
    assert st == B.PRHS_E_WORKSPACE
    return int(re.search(rb"workspace of (\d+) bytes", L.prhs_last_error()).group(1))


def splits(dtype, batch, hq, hkv, d, rows, dense):
    """Splits a unit: partials of d + 2 floats, the outputs rounded up to 256 bytes."""
    n = need(dtype, batch, hq, hkv, d, rows, dense)
    return n // (batch * hq * (d + 2) * 4)


def f32_heads(batch, hq, hkv, d, rows, dense):
    """Query heads of a workgroup of the fp32 kernel on CUS CUs: the launch's rule,
    again."""
    ns, units, g = splits("f32", batch, hq, hkv, d, rows, dense), batch * hkv, hq // hkv
    chunk = -(-(-(-rows // ns)) // 16) * 16
    waves = min(8, -(-chunk // (16 if units * ns < 2 * CUS else 32)))
    gp = 1 if g == 1 else 2 if g == 2 else 4 if g <= 4 else 8
    while gp > 1 and units * ns * waves * -(-g // gp) <= (4 * CUS if gp > 2 else CUS // 2 if ns > 1 or g <= 4 else 0):
        gp //= 2
    return gp


@pytest.mark.parametrize("batch,hkv,d,rows,want", [
    # 129 to 256 units: no split while a workgroup stages the rows
    (129, 1, 128, 2048, 1), (192, 1, 128, 1700, 1), (32, 8, 128, 1989, 1), (31, 8, 64, 2048, 1),
    # a few more units than CUs: unsplit while short, else about 1024 workgroups
    (257, 1, 128, 600, 1), (300, 1, 64, 990, 1), (257, 1, 128, 1142, 4), (40, 8, 128, 1606, 4),
    (264, 1, 64, 1367, 4), (321, 1, 128, 1606, 1), (100, 8, 128, 2000, 1),
    # rows beyond one workgroup: about 1024 workgroups, not a few over a multiple
    # of 512, and at least what staging needs
    (240, 1, 128, 2801, 5), (192, 1, 128, 2953, 5), (32, 8, 128, 8385, 5), (288, 1, 128, 3505, 4), (352, 1, 128, 2122, 2),
    (136, 1, 128, 11811, 7), (72, 8, 128, 3642, 2), (75, 8, 128, 9000, 5),
    # few units: one workgroup a CU for a short stream, two for a long one
    (128, 1, 128, 1400, 2), (2, 8, 128, 65536, 32), (1, 8, 128, 4000, 32), (1, 8, 128, 32768, 64),
])
def test_dense_bf16_splits(batch, hkv, d, rows, want):
    for g in (1, 4):
        assert splits("bf16", batch, hkv * g, hkv, d, rows, True) == want


@pytest.mark.parametrize("batch,hq,hkv,d,rows,dense,want", [
    # short rows unsplit, sets and streams
    (1, 4, 4, 64, 256, False, 1), (64, 1, 1, 64, 257, False, 4), (1, 4, 4, 64, 256, True, 1),
    (1, 16, 1, 64, 128, True, 1), (6, 32, 2, 64, 129, True, 3),
    (40, 16, 1, 128, 450, True, 1), (40, 16, 1, 128, 451, True, 8), (127, 8, 1, 64, 1000, True, 8),
    (128, 8, 1, 64, 1200, True, 1), (128, 8, 1, 64, 1201, True, 8), (160, 1, 1, 128, 1120, True, 1), (39, 2, 1, 128, 257, True, 5),
    # few heads: splits of 32 rows up to 1024 of them, else of 64
    (1, 8, 1, 128, 377, True, 12), (1, 2, 1, 64, 1024, False, 32), (1, 2, 1, 64, 1025, False, 17),
    (12, 16, 1, 128, 1000, True, 16),
    # at most 32 splits once the launch has 256 workgroups
    (1, 8, 8, 128, 8000, False, 32), (2, 16, 8, 128, 8000, True, 32), (32, 8, 8, 128, 3000, True, 4),
])
def test_f32_splits(batch, hq, hkv, d, rows, dense, want):
    assert splits("f32", batch, hq, hkv, d, rows, dense) == want


def size(dtype, batch, hq, hkv, d, rows, dense):
    c, n = kv(dtype, batch, hq, hkv, d, rows), ctypes.c_size_t(0)
    op = B.PRHS_OP_DENSE_ATTN if dense else B.PRHS_OP_SPARSE_ATTN
    assert B.lib().prhs_workspace_size(op, ctypes.byref(c), None, rows, ctypes.byref(n)) == B.PRHS_OK
    return n.value


def test_a_workspace_holds_every_smaller_call():
    assert need("bf16", 1, 8, 8, 128, 2000, False) <= size("bf16", 24, 8, 8, 128, 2000, False)
    rng = random.Random(11)

    def log(a, b):
        return int(math.exp(rng.uniform(math.log(a), math.log(b))))
    for _ in range(20000):
        dtype, dense = rng.choice(["bf16", "f32"]), rng.random() < 0.5
        hkv, g, d = rng.choice([1, 2, 3, 4, 8, 16, 32]), rng.choice([1, 2, 3, 4, 8, 16]), rng.choice([64, 128])
        most, rows = log(1, 400), log(1, 200000)
        batch, r = rng.choice([most, rng.randint(1, most)]), rng.choice([rows, rng.randint(1, rows), log(1, rows)])
        if most * hkv * rows >= 2**31:
            continue
        held = size(dtype, most, hkv * g, hkv, d, rows, dense)
        assert need(dtype, batch, hkv * g, hkv, d, r, dense) <= held, (dtype, dense, hkv, g, d, most, rows, batch, r)
        # and is no multiple of what the largest call takes
        assert held <= max(2.1 * need(dtype, most, hkv * g, hkv, d, rows, dense),
                           (1024 + 2 * most * hkv) * g * (d + 2) * 4 + 256)
