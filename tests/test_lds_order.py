"""What a wave's lanes hand each other through LDS without a barrier is kept in order by a fence, in the device code that is built
(LLVM IR of the kernels, compiled here; no GPU): the compiler sees one lane and may otherwise move its accesses past each other."""
import os
import re
import subprocess

import pytest

from paper_2407_00079_amd import build


def lds_accesses(source, kernel, tmp_path):
    """Of every instantiation of `kernel`: its LDS stores (W) and loads (R) and its fences (F) in order, runs of one kind as one."""
    ll = str(tmp_path / "device.ll")
    subprocess.run([build.HIPCC, *build.FLAGS, "--offload-device-only", "-S", "-emit-llvm", os.path.join(build.CSRC, source), "-o", ll],
                   check=True, capture_output=True)
    found = {}
    for body in re.findall(r"^define [^\n]*amdgpu_kernel.*?^}", open(ll).read(), flags=re.S | re.M):
        name = re.search(r"@(\w+)\(", body).group(1)
        if kernel not in name:
            continue
        kinds = ""
        for line in body.splitlines():
            if re.match(r"\s+fence ", line):
                kinds += "F"
            elif re.search(r"\bstore\b.*, ptr addrspace\(3\)", line):
                kinds += "W"
            elif re.search(r"= load\b.*, ptr addrspace\(3\)", line):
                kinds += "R"
        found[name] = re.sub(r"(.)\1+", r"\1", kinds)
    return found


@pytest.mark.parametrize("kernel", ["attn_narrow_classes_kernel", "attn_narrow_list_kernel"])
def test_blocks_of_keys_turned_in_lds(kernel, tmp_path):
    """A block is put down, fragments of it are read, and the place is free for the next block or the wave's output.  (What follows
    the loop is behind a barrier and may be laid out in any order.)"""
    found = lds_accesses("attn_narrow.hip", kernel, tmp_path)
    assert len(found) == 5                        # fp32; bf16 of two head sizes with 16 and 32 rows
    for name, kinds in found.items():
        assert kinds.startswith("WFRF"), (name, kinds)
