"""The lengths of wide_util.py take the forms that they are listed with (csrc/host_plan.cpp; no GPU)."""
import os
import subprocess

from paper_2407_00079_amd import workloads as W

from wide_util import CUT, HEADS, WHOLE

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_2407_00079_amd", "csrc")

DRIVER = r"""
#include <cstdio>
#include "host_plan.h"
int main() {
  int Hq, Hkv, D, dtype;
  int32_t P, C;
  while (std::scanf("%d %d %d %d %d %d", &Hq, &Hkv, &D, &dtype, &P, &C) == 6) {
    const mc_attn_params p{Hq, Hkv, D, 16, 1 << 20, dtype, 0.f};
    mc::host::ClassPlan whole;
    mc::host::AutoLayout room;
    if (!mc::host::plan_classes(&p, &P, &C, 1, 0, &whole) || !mc::host::auto_layout(&p, &P, &C, 1, &room) || !room.by_classes) return 1;
    std::printf("%d %d %d %d %d\n", whole.narrow_wgs, whole.classes.rows, room.plan.narrow_wgs, room.plan.classes.rows, room.plan.most_pieces);
  }
}
"""


def test_forms_of_the_wide_shapes(tmp_path):
    src, exe = str(tmp_path / "driver.cpp"), str(tmp_path / "driver")
    with open(src, "w") as f:
        f.write(DRIVER)
    subprocess.run(["g++", "-O1", "-std=c++17", "-Wall", "-I", os.path.join(ROOT, "include"), "-I", CSRC, "-o", exe, src,
                    os.path.join(CSRC, "host_plan.cpp")], check=True)
    lines = [" ".join(str(x) for x in (*HEADS, D, int(dtype == W.F32), *prefix, *new)) for _, dtype, D, prefix, new in WHOLE + CUT]
    out = subprocess.run([exe], input="\n".join(lines) + "\n", capture_output=True, text=True, check=True).stdout.splitlines()
    assert len(out) == len(lines)
    for i, (shape, line) in enumerate(zip(WHOLE + CUT, out)):
        narrow, rows, narrow_room, rows_room, pieces = (int(x) for x in line.split())
        if i < len(WHOLE):
            assert narrow == 0 and rows == shape[0], shape
        else:
            assert narrow == 0 and narrow_room == 0 and rows_room == shape[0] and pieces > 1, shape
