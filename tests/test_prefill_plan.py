"""How prefill launches divide their prompts (prefill_plan.h), on the host: the
header compiled into a small program and asked."""

import math
import os
import random
import shutil
import subprocess

import pytest

from paper_2602_08329_amd import build

HERE = os.path.dirname(os.path.abspath(__file__))

# launches of every form of the kernel on 256 CUs: waves of w queries, ns key
# sides, d, paged, and batch, query heads and T under the window of WINDOW
FORMS = [
    (16, 1, 128, False, 1, 64, 113), (16, 1, 128, True, 2, 64, 173),
    (32, 1, 128, False, 3, 60, 255), (32, 1, 128, True, 5, 24, 321),
    (32, 2, 128, False, 1, 60, 257), (32, 2, 128, True, 3, 24, 257),
    (32, 4, 128, False, 2, 4, 300), (32, 4, 128, True, 2, 8, 777),
    (16, 1, 64, False, 2, 64, 265), (16, 1, 64, True, 1, 60, 97),
    (32, 1, 64, False, 4, 64, 300), (32, 1, 64, True, 3, 48, 300),
    (32, 2, 64, False, 3, 24, 384), (32, 2, 64, True, 1, 48, 330),
    (32, 4, 64, False, 1, 4, 500), (32, 4, 64, True, 1, 48, 300),
    # blocks for every CU eight times over: 256 queries whatever else
    (32, 1, 64, True, 8, 64, 1000),
]
WINDOW = dict(psaw=(2, 0.6, 1.0), layer=3, n_layers=4, sink=5)


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


# ---------------------------------------------------------------- the plan

def shape(T, units, d=128, paged=0, psaw=0, factor=0.0, sink=4, cus=256):
    return f"{T} {units} {d} {paged} {psaw} {factor:.17g} {sink} {cus}"


def test_plans_cover_their_prompts(ask):
    rng = random.Random(5)
    shapes = []
    for _ in range(3000):
        T = int(math.exp(rng.uniform(0, math.log(200000))))
        units = int(math.exp(rng.uniform(0, math.log(3000))))
        psaw = rng.randrange(2)
        shapes.append((T, units, rng.choice([64, 128]), rng.randrange(2), psaw, rng.random() * 0.95 * psaw,
                       rng.choice([0, 4, 300]), rng.choice([256, 256, 32, 0])))
    for s, r in zip(shapes, ask(["plan " + shape(*s) for s in shapes])):
        w, ns, qb, qf, n = map(int, r)
        assert (w, ns) in ((16, 1), (32, 1), (32, 2), (32, 4)), s
        most = w * (12 if w == 16 else 8) // ns   # queries of a workgroup's waves
        assert 0 < qb <= most and 0 < qf <= most and qb % w == 0 and qf % w == 0, (s, r)
        assert qf + (n - 1) * qb >= s[0] and (n == 1 or qf + (n - 2) * qb < s[0]), (s, r)


def test_work_of_a_plan_is_bounded(ask):
    # every layer of a model asks for one: long prompts of few units, whose
    # blocks are many, cost no multiple of what a prompt of 48 blocks does
    short, *long = (float(r[0]) for r in ask(
        ["time " + shape(*a) for a in ((2900, 4), (24000, 4), (131072, 1), (131072, 1, 64, 1, 1, 0.3))]))
    assert max(long) <= 3 * short, (short, long)


def test_left_over_queries_of_a_long_prompt_come_last(ask):
    # 64 blocks for 32 CUs an XCD; and queries, not key sides, where two a CU follow
    assert [r[:4] for r in ask(["plan " + shape(12197, 8), "plan " + shape(11000, 8),
                                "plan " + shape(10611, 8, 128, 0, 1, 0.2)])] == [["16", "1", "192", "192"]] * 3


def test_forms_are_those_the_launches_take(ask):
    l_s, phi, alpha = WINDOW["psaw"]
    factor = 1 - phi ** (alpha * (WINDOW["layer"] + 1 - l_s) / (WINDOW["n_layers"] - l_s))
    got = ask(["plan " + shape(T, batch * hq, d, int(paged), 1, factor, WINDOW["sink"])
               for _, _, d, paged, batch, hq, T in FORMS])
    for form, r in zip(FORMS, got):
        assert tuple(map(int, r[:2])) == form[:2], (form, r)
    assert {f[:4] for f in FORMS} == {(w, ns, d, paged) for w, ns in ((16, 1), (32, 1), (32, 2), (32, 4))
                                      for d in (64, 128) for paged in (False, True)}
