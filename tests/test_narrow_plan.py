"""When an attention launch takes the narrow form and the classes it is described with then (csrc/host_plan.cpp; no GPU):
every row tile of every request once, and the same decision for prepared lists."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2407_00079_amd", "csrc")

DRIVER = r"""
#include <cstdio>
#include <vector>
#include "host_plan.h"
int main() {
  int Hq, Hkv, D, dtype, batch;
  long long room;
  if (std::scanf("%d %d %d %d %lld %d", &Hq, &Hkv, &D, &dtype, &room, &batch) != 6) return 1;
  std::vector<int32_t> P(batch), C(batch);
  for (auto& x : P) if (std::scanf("%d", &x) != 1) return 1;
  for (auto& x : C) if (std::scanf("%d", &x) != 1) return 1;
  const mc_attn_params p{Hq, Hkv, D, 16, 1 << 20, dtype, 0.f};
  mc::host::ClassPlan plan;
  if (!mc::host::plan_classes(&p, P.data(), C.data(), batch, room, &plan)) return 2;
  const int32_t form = mc::host::list_form(&p, P.data(), C.data(), batch, 0, mc::host::count_items(&p, C.data(), batch));
  std::printf("%d %d %d %lld", plan.narrow_wgs, plan.narrow_pieces, form == mc::host::kListNarrow || form == mc::host::kListNarrowLeast, (long long)plan.part_rows);
  for (int i = 0; plan.narrow_wgs > 0 && i < plan.narrow.n; ++i) {
    const mc::AttnClass& k = plan.narrow.c[i];
    std::printf(" %d %d %d %d %d %d %d %d %d", plan.narrow.first[i], k.req, k.q_off, k.prefix, k.chunk, k.tile_lo, k.tile_hi, k.pieces,
                k.part_base);
  }
  return 0;
}
"""


@pytest.fixture(scope="module")
def driver(tmp_path_factory):
    d = tmp_path_factory.mktemp("narrow")
    src, exe = str(d / "driver.cpp"), str(d / "driver")
    with open(src, "w") as f:
        f.write(DRIVER)
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-fsanitize=address,undefined", "-I", os.path.join(ROOT, "include"), "-I", CSRC,
                    "-o", exe, src, os.path.join(CSRC, "host_plan.cpp")], check=True)
    return exe


# the last columns: with no room for partial results, and most pieces with room for 64 parts of every row (0: another form)
@pytest.mark.parametrize("Hq,Hkv,D,dtype,prefix,new,without,pieces", [
    (4, 1, 64, 1, [256], [128], True, 1),                     # a few short row tiles: no merge to pay for
    (64, 8, 128, 0, [1023], [4], True, 1),
    (12, 3, 128, 0, [999, 1, 0], [130, 0, 257], True, 1),
    (64, 8, 128, 0, [131056], [16], True, 0),                 # bound by the memory
    (8, 1, 128, 0, [123051], [4], True, 64),
    (16, 16, 128, 0, [300, 20], [16, 3], True, 1),            # 16 rows a workgroup
    (16, 16, 128, 0, [300, 20], [17, 3], True, 1),            # one request has more
    (4, 1, 128, 0, [24530, 300], [118, 20], True, 16),        # pieces in proportion
    (64, 8, 128, 0, [8192], [8192], False, 0),                # many rounds of full row tiles
    (64, 8, 128, 0, [6144, 6144], [811, 328], False, 0),
    (64, 8, 128, 0, [16384] * 16, [16] * 16, False, 0),       # bound by the memory: row tiles would read their keys apart
    (64, 8, 128, 0, [20], [16], False, 0),                    # one key tile
    (8, 2, 64, 1, [4090], [6], True, 64),                     # fp32: up to 4096 keys, of a piece
    (8, 2, 64, 1, [4091], [6], False, 24),
    (8, 2, 128, 0, [200] * 63, [7] * 63, True, 1),            # as many requests as there are classes
])
def test_the_narrow_form_is_taken_where_it_is_sooner(driver, Hq, Hkv, D, dtype, prefix, new, without, pieces):
    G = Hq // Hkv
    rows = 16 if dtype or max(new) * G <= 16 else 32
    for room, most in ((0, 1 if without else 0), (64 * sum(new) * Hq, pieces)):
        line = " ".join(str(x) for x in [Hq, Hkv, D, dtype, room, len(prefix), *prefix, *new])
        v = [int(x) for x in subprocess.run([driver], input=line, capture_output=True, text=True, check=True).stdout.split()]
        assert (v[1] if v[0] > 0 else 0) == most and v[2] == without
        wg, parts, seen = 0, 0, set()
        for at in range(4, len(v), 9):
            first, req, q_off, p, c, lo, hi, cut, base = v[at:at + 9]
            assert (first, q_off, p, c, lo) == (wg, sum(new[:req]), prefix[req], new[req], 0)
            assert hi == -(-c * G // rows) - 1 and req not in seen and 1 <= cut <= v[1]
            seen.add(req)
            wg += (hi + 1) * Hkv * cut
            if cut > 1:                                       # [part_base, part_base + pieces rows): one block after another
                assert base == parts
                parts += cut * c * Hq
        assert wg == v[0] and (not most or seen == {r for r in range(len(new)) if new[r] > 0})
        assert parts <= v[3]                                  # no more room than the plan it replaces
