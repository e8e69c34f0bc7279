"""As test_lds_order.py, for the narrow kernels whose workgroups take a share of the columns (fp32 and head_dim 128 in two and four
shares, head_dim 64 in two)."""
import re

import pytest

from test_lds_order import kernels_of


@pytest.mark.parametrize("kernel", ["attn_narrow_shared_classes_kernel", "attn_narrow_shared_list_kernel"])
def test_blocks_of_keys_turned_in_lds(kernel, tmp_path):
    found = kernels_of("attn_narrow.hip", kernel, tmp_path)
    assert len(found) == 8                        # fp32 2; bf16 16 and 32 rows, 128 in 2 and 4 shares, 64 in 2
    for name, lines in found.items():
        kinds = "".join("F" if re.match(r"\s+fence ", line) else "W" if re.search(r"\bstore\b.*, ptr addrspace\(3\)", line)
                        else "R" if re.search(r"= load\b.*, ptr addrspace\(3\)", line) else "" for line in lines)
        assert re.sub(r"(.)\1+", r"\1", kinds).startswith("WFRF"), (name, kinds)
