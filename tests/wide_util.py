"""Lengths whose attention takes the kernels of 128- and 256-row workgroups (csrc/attn_prefill.hip, attn_prefill_bf16.hip), which
the narrow form leaves to larger calls.  tests/test_wide_shapes.py asks the plan for the cut ones; GPU tests ask a prepared list."""
from paper_2407_00079_amd import binding as B
from paper_2407_00079_amd import workloads as W

# mc_attn_plan.reserved of a list of whole rows -> rows of its workgroups; the narrow form's marks are not among them
WIDE_LIST = {0: 256, 0x4d434631: 128, 0x4d434632: 128, 0x4d434633: 128}

# rows of a workgroup, dtype, head_dim, prefix, new: whole rows, 64/8 heads
WHOLE = [(128, W.BF16, 128, [2000], [130]), (256, W.BF16, 128, [2000], [600]), (128, W.BF16, 64, [2000], [130]),
         (256, W.BF16, 64, [900], [600]), (128, W.F32, 64, [700], [200]), (256, W.F32, 64, [700], [1000])]

# the same where a one-shot call has room for partial results: its row tiles, or the last of them, are cut
CUT = [(128, W.BF16, 128, [2000], [130]), (256, W.BF16, 128, [1000], [1100]), (128, W.BF16, 64, [2000], [130]),
       (256, W.BF16, 64, [2000], [1100]), (128, W.F32, 64, [700], [200]), (256, W.F32, 64, [700], [1100])]

HEADS = (64, 8)


def with_short_requests(prefix, new, n=64):
    """More requests than an argument describes: the call takes a list, and lists of so many are not weighed against the narrow
    form."""
    return list(prefix) + [0] * n, list(new) + [1] * n


def rows_of_list(params, prefix, new, workspace) -> int:
    """Rows of a workgroup of the batch's prepared list; fails for the narrow form.  (What runs of whole rows takes these.)"""
    return WIDE_LIST[B.mc_prefill_attn_prepare(params, prefix, new, 0, workspace).reserved]
