"""How prefill launches divide their prompts (prefill_plan.h), on the host: the
header compiled into a small program and asked."""

import os
import shutil
import subprocess

import pytest

from paper_2602_08329_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))


@pytest.fixture(scope="module")
def ask(tmp_path_factory):
    cc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    exe = str(tmp_path_factory.mktemp("plan") / "probe")
    subprocess.run([cc, "-O2", *(f for f in build.FLAGS if f not in ("-O3", "-fPIC")), "-I", build.CSRC,
                    "-I", build.INCLUDE, "-o", exe, os.path.join(HERE, "prefill_plan_probe.hip")],
                   check=True, capture_output=True, text=True)

    def run(lines):
        r = subprocess.run([exe], input="\n".join(lines) + "\n", capture_output=True, text=True,
                           timeout=120, check=True)
        out = [ln.split() for ln in r.stdout.splitlines()]
        assert len(out) == len(lines)
        return out
    return run


# ---------------------------------------------------------------- block order

@pytest.mark.parametrize("units,nqb,group", [
    (8, 5, 1), (40, 9, 5), (40, 9, 3), (64, 1, 8), (64, 7, 4), (72, 3, 9), (24, 4, 2), (12, 6, 1),
    (1, 9, 1), (7, 3, 1)])
def test_every_block_once_longest_first_in_its_group(ask, units, nqb, group):
    (line,) = ask([f"order {units} {nqb} {group}"])
    seq = [tuple(map(int, x.split(":"))) for x in line]
    assert sorted(seq) == [(u, q) for u in range(units) for q in range(nqb)]
    lists = [seq[x::8] for x in range(8)] if units % 8 == 0 else [seq]
    per = units // 8 if units % 8 == 0 else units
    for x, xcd in enumerate(lists):   # what one XCD takes, in order
        if units % 8 == 0:
            assert {u for u, _ in xcd} == set(range(x * per, (x + 1) * per))
        size = group if units % 8 == 0 else per
        for g0 in range(0, per, size):
            part = xcd[g0 * nqb:min(g0 + size, per) * nqb]
            assert {u - (x * per if units % 8 == 0 else 0) for u, _ in part} == set(range(g0, min(g0 + size, per)))
            blocks = [q for _, q in part]
            assert blocks == sorted(blocks, reverse=True)


def test_groups_hold_enough_blocks_to_end_a_launch_evenly(ask):
    cases = [(per, nqb) for per in range(1, 41) for nqb in (1, 2, 5, 9, 16, 33, 48, 97, 200, 1000)]
    got = [int(r[0]) for r in ask([f"group {per} {nqb} 256" for per, nqb in cases])]
    for (per, nqb), g in zip(cases, got):
        assert 1 <= g <= per
        groups = -(-per // g)
        last = per - (groups - 1) * g
        # four rounds of the XCD's 32 CUs a group, the last up to its share less
        assert g == per or g * nqb >= 128
        assert groups == 1 or last >= g - groups + 1
        # and no more than it takes
        assert g * nqb < 2 * (128 + nqb) or g == 1
