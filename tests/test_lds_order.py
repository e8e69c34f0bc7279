"""What lanes and waves hand each other through LDS without a barrier is kept in order by fences, in the device code that is built
(LLVM IR of the kernels, compiled here; no GPU): the compiler sees one lane and may otherwise move its accesses past each other."""
import os
import re
import subprocess

import pytest

from paper_2407_00079_amd import build


def kernels_of(source, kernel, tmp_path):
    """The IR of every instantiation of `kernel`: name -> lines."""
    ll = str(tmp_path / "device.ll")
    subprocess.run([build.HIPCC, *build.FLAGS, "--offload-device-only", "-S", "-emit-llvm", os.path.join(build.CSRC, source), "-o", ll],
                   check=True, capture_output=True)
    bodies = re.findall(r"^define [^\n]*amdgpu_kernel.*?^}", open(ll).read(), flags=re.S | re.M)
    named = {re.search(r"@(\w+)\(", body).group(1): body.splitlines() for body in bodies}
    return {name: lines for name, lines in named.items() if kernel in name}


@pytest.mark.parametrize("kernel", ["attn_narrow_classes_kernel", "attn_narrow_list_kernel"])
def test_blocks_of_keys_turned_in_lds(kernel, tmp_path):
    """A block is put down, fragments of it are read, and the place is free for the next block or the wave's output.  (What follows
    the loop is behind a barrier and may be laid out in any order.)"""
    found = kernels_of("attn_narrow.hip", kernel, tmp_path)
    assert len(found) == 5                        # fp32; bf16 of two head sizes with 16 and 32 rows
    for name, lines in found.items():
        kinds = ""                                # LDS stores and loads and fences in order, runs of one kind as one
        for line in lines:
            if re.match(r"\s+fence ", line):
                kinds += "F"
            elif re.search(r"\bstore\b.*, ptr addrspace\(3\)", line):
                kinds += "W"
            elif re.search(r"= load\b.*, ptr addrspace\(3\)", line):
                kinds += "R"
        kinds = re.sub(r"(.)\1+", r"\1", kinds)
        assert kinds.startswith("WFRF"), (name, kinds)


def test_digests_of_other_waves(tmp_path):
    """The chain reads digests that other waves of its workgroup put down: released by the count it has seen, acquired behind it."""
    found = kernels_of("prefix_hash.hip", "prefix_pour_kernel", tmp_path)
    assert len(found) == 2                        # tables in the kernel argument and in memory
    for name, lines in found.items():
        assert any("atomicrmw add ptr addrspace(3)" in line and 'syncscope("workgroup") release' in line for line in lines), name
        reads = [i for i, line in enumerate(lines) if re.search(r"= load .*, ptr addrspace\(3\)", line)]
        counts, digests = [i for i in reads if " i32," in lines[i]], [i for i in reads if " i64," in lines[i]]
        assert counts and digests and len(counts) + len(digests) == len(reads)
        assert all('load atomic i32' in lines[i] and 'syncscope("workgroup") monotonic' in lines[i] for i in counts), name
        for i in digests:                         # between the count and the digests, in the same block
            behind = next(line for line in reversed(lines[:i]) if re.search(r"^\S+:|fence|= load|\bstore\b|atomicrmw", line))
            assert re.match(r'\s+fence syncscope\("workgroup"\) acquire', behind), (name, behind)
