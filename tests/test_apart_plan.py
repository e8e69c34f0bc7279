"""Whole-row attention as two launches, requests of few rows and then the others (csrc/host_plan.cpp: plan_apart; no GPU)."""
import os
import random
import subprocess

import pytest

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


def ask(exe, batches):
    text = "".join(" ".join(str(x) for x in [*b[:4], len(b[4]), *b[4], *b[5]]) + "\n" for b in batches)
    res = subprocess.run([exe], input=text, capture_output=True, text=True, timeout=300)
    assert res.returncode == 0 and res.stderr == "", res.stderr[-2000:]
    out = [line.split() for line in res.stdout.splitlines()]
    assert len(out) == len(batches)
    return out


@pytest.mark.skipif(not os.path.exists(CLANG), reason="needs clang's MemorySanitizer")
def test_no_choice_reads_what_no_plan_has_written(tmp_path):
    """A first launch whose plan is not narrow has no narrow classes to look at."""
    exe = build(tmp_path, "-O0", "-g", "-fsanitize=memory", cxx=CLANG)
    rng = random.Random(5)
    launches = [what for what, *_ in ask(exe, [draw(rng) for _ in range(1500)])]
    assert launches.count("two") > 20 and launches.count("one") > 20


def test_the_choice_of_two_launches_uses_no_heap(tmp_path):
    """mc_prefill_attn_paged_noalloc plans with these functions and promises to allocate nothing, on the host heap either."""
    rng = random.Random(6)
    # one launch by the narrow or a wide form, or two: no batch here weighs 64-row workgroups
    batches = [b for b in (draw(rng) for _ in range(6000)) if b[3] == 1] + [(64, 8, 128, 0, [6000, 0], [3, 900])]
    out = ask(build(tmp_path, "-O2", "-DCOUNT_NEWS"), batches)
    assert sum(what == "two" for what, *_ in out) > 20
    assert [b for b, (_, _, by_apart) in zip(batches, out) if by_apart != "0"] == []
