"""Whole-row attention as two launches, requests of few rows and then the others (csrc/host_plan.cpp: plan_apart; no GPU)."""
import os
import random
import subprocess

import pytest

from paper_2407_00079_amd import binding as B
from test_class_plan import launch_end

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2407_00079_amd", "csrc")
CLANG = "/opt/rocm/llvm/bin/clang++"

HEADS = [(64, 8, 128, 0), (64, 8, 64, 0), (16, 2, 128, 0), (12, 3, 128, 0), (16, 16, 64, 1), (64, 8, 64, 1), (8, 1, 128, 0)]


def build(tmp, *flags, cxx="g++"):
    exe = str(tmp / "apart_plan_driver")
    subprocess.run([cxx, "-std=c++17", "-Wall", *flags, "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-o", exe,
                    os.path.join(ROOT, "tests", "apart_plan_driver.cpp"), os.path.join(CSRC, "host_plan.cpp")], check=True)
    return exe


def draw(rng):
    """A batch of some requests with few new tokens and some with many, which is where two launches are weighed."""
    n = rng.randint(2, 12)
    new = [rng.choice((0, 1, 3, rng.randint(1, 40), int(2 ** rng.uniform(5, 12)))) for _ in range(n)]
    prefix = [rng.choice((0, rng.randrange(60), int(2 ** rng.uniform(6, 16)))) for _ in range(n)]
    return (*rng.choice(HEADS), prefix, new)


def lines_of(exe, batches, *args):
    text = "".join(" ".join(str(x) for x in [*b[:4], len(b[4]), *b[4], *b[5]]) + "\n" for b in batches)
    res = subprocess.run([exe, *args], input=text, capture_output=True, text=True, timeout=300)
    assert res.returncode == 0 and res.stderr == "", res.stderr[-2000:]
    lines = res.stdout.splitlines()
    assert len(lines) == len(batches)
    return lines


def ask(exe, batches):
    out = [line.split() for line in lines_of(exe, batches)]
    assert all(line[5] == "1" for line in out)
    return out


@pytest.mark.skipif(not os.path.exists(CLANG), reason="needs clang's MemorySanitizer")
def test_no_choice_reads_what_no_plan_has_written(tmp_path):
    """A first launch whose plan is not narrow has no narrow classes to look at."""
    exe = build(tmp_path, "-O0", "-g", "-fsanitize=memory", cxx=CLANG)
    rng = random.Random(5)
    launches = [what for what, *_ in ask(exe, [draw(rng) for _ in range(1500)])]
    assert launches.count("two") > 20 and launches.count("one") > 20


def test_planning_uses_no_heap(tmp_path):
    """mc_prefill_attn_paged_noalloc plans with these functions and promises to allocate nothing, on the host heap either."""
    rng = random.Random(6)
    batches = [draw(rng) for _ in range(3000)] + [(64, 8, 128, 0, [6000, 0], [3, 900]), (64, 8, 128, 0, [8192], [192])]
    out = ask(build(tmp_path, "-O2", "-DCOUNT_NEWS"), batches)
    assert sum(what == "two" for what, *_ in out) > 20 and sum(line[3] == "64" for line in out) > 20
    assert [b for b, (_, by_classes, by_apart, *_) in zip(batches, out) if (by_classes, by_apart) != ("0", "0")] == []


def pairs_end(Hq, Hkv, D, dtype, prefix, new):
    """End of a launch of 64-row workgroups, the quarters of eight items of the list after the other, each quarter's workgroups
    where they go."""
    launch, fixed, tile = (2.1, 4.6, 0.44) if D == 128 else (1.5, 3.2, 0.36)
    G = Hq // Hkv
    items = B.mc_prefill_attn_plan(B.attn_params(Hq, Hkv, D, 16, 1 << 20, "bf16"), prefix, new, 0)
    rest = len(items) % 8
    order = [(items[at + i], part) for at in range(0, len(items) - rest, 8) for part in range(4) for i in range(8)]
    order += [(item, part) for part in range(4) for item in items[len(items) - rest:]]

    def us(item, part):
        row0 = item[2] + 64 * part
        P, C = prefix[item[0]], new[item[0]]
        return fixed + tile * -(-(P + min(C - 1, (row0 + 63) // G) + 1) // 64) if row0 < C * G else 1.0
    return launch + launch_end([us(*w) for w in order])


def test_64_row_workgroups_are_weighed_by_where_those_of_the_list_go(tmp_path):
    """Heads that fill the eight lists evenly and heads that do not, requests with the same keys, requests without new tokens."""
    rng = random.Random(8)
    batches = [(*rng.choice([h for h in HEADS if h[3] == 0] + [(40, 40, 128, 0), (4, 1, 64, 0), (24, 8, 128, 0)]),
                [rng.choice((2600, 9000, rng.randrange(30000))) for _ in range(n)], [rng.choice((0, 200, rng.randint(1, 900))) for _ in range(n)])
               for n in (rng.choice((1, 2, 3, 6)) for _ in range(1200))]
    out = ask(build(tmp_path, "-O2"), batches)
    pairs = [(b, float(line[4])) for b, line in zip(batches, out) if line[3] == "64"]
    assert len(pairs) > 150 and {b[1] for b, _ in pairs} >= {8, 2, 3, 1}
    for b, ends in pairs:
        assert ends == pytest.approx(pairs_end(*b), rel=1e-6), b


FORMS = {0: 256, 0x4d434631: 128, 0x4d434632: 128, 0x4d434633: 128, 0x4d434636: 64}       # rows of the second launch's workgroups


def test_two_launches_and_their_list_cover_every_row_tile_once(tmp_path):
    """Under AddressSanitizer and UBSan: the classes of both launches, at the rows of the whole batch in q and out, the list of the
    same two launches, and its mark."""
    exe = build(tmp_path, "-O1", "-fsanitize=address,undefined", "-fno-sanitize-recover=all")
    rng = random.Random(11)
    batches = [draw(rng) for _ in range(4000)]
    # (of test_gpu_apart.py)
    batches += [(64, 8, 128, 0, [6000, 0], [3, 900]), (64, 8, 128, 0, [0, 7001], [1100, 33]), (64, 8, 128, 0, [17, 5, 12000, 3], [900, 0, 3, 5]),
                (16, 2, 128, 0, [108, 14659, 1947], [2942, 299, 183]), (64, 8, 64, 0, [12007, 17, 0, 3], [17, 600, 0, 5])]
    forms, leasts = set(), set()
    for (Hq, Hkv, D, dtype, prefix, new), line in zip(batches, lines_of(exe, batches, "two")):
        if line == "":
            continue
        (at,), few, many, mark, items = ([int(x) for x in part.split()] for part in line.split("|"))
        G = Hq // Hkv
        seen = {}
        for launch, (rows, *classes) in enumerate((few, many)):
            wg = 0
            for i in range(0, len(classes), 8):
                first, r, q_off, P, C, lo, hi, pieces = classes[i:i + 8]
                assert (q_off, P, C, pieces, first) == (sum(new[:r]), prefix[r], new[r], 1, wg)
                assert (0 < C <= at) if launch == 0 else C > at
                wg += (hi - lo + 1) * Hkv
                for t in range(lo, hi + 1):
                    assert (r, t) not in seen
                    seen[r, t] = rows
        assert set(seen) == {(r, t) for r, C in enumerate(new) for t in range(-(-C * G // (few if C <= at else many)[0]))}
        packed, read, small, n_few, shares, least, form, want_shares = mark
        assert packed >> 16 == 0x4d44 and (read, small, shares) == (1, 0, want_shares)
        assert few[0] == (16 if least or dtype == 1 else 32) and many[0] == FORMS[form]
        items = [tuple(items[i:i + 4]) for i in range(0, len(items), 4)]
        whole = B.mc_prefill_attn_plan(B.attn_params(Hq, Hkv, D, 16, 1 << 20, ("bf16", "f32")[dtype]), prefix, new, 0)
        assert len(set(items)) == len(items) and set(items) == set(whole)
        assert all(new[r] <= at for r, *_ in items[:n_few]) and all(new[r] > at for r, *_ in items[n_few:])
        if least:
            assert dtype == 1 or max(new[r] for r, *_ in items[:n_few]) * G <= 16          # an item is one row tile
        forms.add(form)
        leasts.add((dtype, least))
    assert forms >= {0, 0x4d434633, 0x4d434636} and leasts == {(0, 0), (0, 1), (1, 1)}
