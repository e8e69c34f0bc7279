"""GPU parity of the narrow form of the attention kernels (csrc/attn_narrow.hip: waves share out the keys of 32 or, fp32, 16
rows), at the edges of its rows, key blocks and waves, against the oracle; whole rows are the same bits however the call is
driven.  The pools hold NaN behind every request's last key."""
import numpy as np
import pytest
import torch

from paper_2407_00079_amd import binding as B
from paper_2407_00079_amd import workloads as W

from gpu_util import TOL, DeviceCase, check_close

pytestmark = pytest.mark.gpu

NARROW, LEAST = 0x4d434634, 0x4d434635         # mc_attn_plan.reserved of a list that is launched so; no request has more than 16 rows

# dtype, Hq, Hkv, D, prefix, new
CASES = [(W.BF16, 8, 1, 128, [keys - 4], [4]) for keys in (65, 95, 96, 97, 255, 256, 257, 288, 289, 511, 513, 545)]    # 32 rows; blocks per wave
CASES += [(W.BF16, 8, 2, 64, [keys - 9], [9]) for keys in (66, 256, 257, 300)]                                       # 36 rows: a row tile of 4
CASES += [(W.F32, 4, 1, 64, [keys - 5], [5]) for keys in (67, 96, 255, 256, 257, 290)]                               # 20 rows: 16 and 4
CASES += [
    (W.BF16, 8, 1, 128, [300], [1]),                          # 8 rows
    (W.BF16, 4, 1, 128, [255, 900, 0], [1, 4, 3]), (W.BF16, 16, 16, 128, [285], [16]), (W.BF16, 16, 16, 64, [77, 640], [16, 1]),
    (W.BF16, 16, 16, 128, [285, 30], [17, 16]), (W.F32, 8, 2, 64, [100, 513], [4, 1]),       # 16 rows, and one more
    (W.BF16, 16, 1, 128, [70], [2]),                          # exactly a row tile of 16 heads a group
    (W.BF16, 64, 8, 128, [1023], [33]),                       # 264 rows: more than one item of the list, the last of 8 rows
    (W.BF16, 12, 3, 128, [999, 1, 0], [130, 0, 257]),         # three heads, an empty request, no prefix: row tiles of one to five key tiles
    (W.BF16, 16, 16, 64, [700, 81], [70, 1]),                 # one head a group
    (W.F32, 12, 3, 64, [500, 31, 0], [17, 100, 40]),
    (W.F32, 16, 16, 64, [4000], [3]),                         # just inside what fp32 takes
]


@pytest.mark.parametrize("q_scale", [1.0, 8.0])               # 8: references that are raised many times
@pytest.mark.parametrize("dtype,Hq,Hkv,D,prefix,new", CASES)
def test_narrow_form_matches_oracle(oracle, dtype, Hq, Hkv, D, prefix, new, q_scale):
    print(f"narrow case {dtype} Hq={Hq} Hkv={Hkv} D={D} prefix={prefix} new={new} q_scale={q_scale}", flush=True)
    pages = sum(-(-(p + c) // 16) for p, c in zip(prefix, new)) + 5
    case = W.make_attn_case(95, dtype, Hq, Hkv, D, 16, prefix, new, pages, q_scale=q_scale)
    dc = DeviceCase(case)
    plan_ws = torch.empty_like(dc.workspace)
    plan = B.mc_prefill_attn_prepare(dc.params, prefix, new, 0, plan_ws)
    assert plan.reserved == (LEAST if max(new) * (Hq // Hkv) <= 16 else NARROW)
    args = (dc.q, dc.k_pool, dc.v_pool, dc.block_tables)
    ref_out, ref_lse, _ = oracle.case_full(case)
    first = None
    for call in (lambda: B.mc_prefill_attn_run(dc.params, plan, *args, dc.out, dc.lse, plan_ws), dc.run,
                 lambda: B.mc_prefill_attn_paged_noalloc(dc.params, *args, prefix, new, dc.out, dc.lse)):
        dc.out.fill_(float("nan"))
        dc.lse.fill_(float("nan"))
        call()
        out, lse = dc.result()
        check_close(out, ref_out, dtype, "narrow")
        assert np.abs(lse - ref_lse).max() <= TOL[dtype]["lse_abs"]
        bits = dc.out.clone(), dc.lse.clone()
        first = first or bits
        assert torch.equal(bits[0], first[0]) and torch.equal(bits[1], first[1])


# one call with room for partial results: narrow row tiles cut into pieces, and (the second half) shapes whose row tiles of 128
# and of 256 rows are cut all the same
PIECES = [
    (W.BF16, 8, 1, 128, [12000], [2]), (W.BF16, 16, 16, 64, [5000, 90], [16, 3]),
    (W.BF16, 8, 1, 128, [9000], [4]), (W.BF16, 4, 1, 128, [5531, 300], [70, 20]), (W.BF16, 8, 1, 128, [15000, 0, 63], [1, 9, 5]),
    (W.BF16, 16, 2, 64, [6001], [17]), (W.BF16, 12, 3, 128, [4100, 64], [33, 1]),
    (W.F32, 8, 2, 64, [4091], [6]), (W.F32, 4, 1, 64, [9000, 17], [9, 40]), (W.F32, 16, 16, 64, [2100], [17]),
    (W.BF16, 8, 2, 128, [401, 10503], [70, 1]), (W.BF16, 4, 1, 128, [250, 6614, 142], [80, 9, 76]), (W.BF16, 64, 8, 128, [7, 7908], [370, 2]),
    (W.BF16, 64, 8, 64, [10515, 118], [2, 120]), (W.BF16, 64, 8, 64, [53, 1495], [419, 21]), (W.F32, 64, 8, 64, [68, 304], [147, 45]),
    (W.F32, 64, 8, 64, [103, 704], [180, 33]),
]


@pytest.mark.parametrize("dtype,Hq,Hkv,D,prefix,new", PIECES)
def test_cut_row_tiles_match_oracle(oracle, dtype, Hq, Hkv, D, prefix, new):
    print(f"cut case {dtype} Hq={Hq} Hkv={Hkv} D={D} prefix={prefix} new={new}", flush=True)
    pages = sum(-(-(p + c) // 16) for p, c in zip(prefix, new)) + 5
    case = W.make_attn_case(96, dtype, Hq, Hkv, D, 16, prefix, new, pages, q_scale=4.0)
    dc = DeviceCase(case)
    need = B.mc_prefill_attn_auto_workspace_bytes(dc.params, prefix, new)
    assert need > B.mc_prefill_attn_workspace_bytes(dc.params, case.batch, case.total_new)
    # the workspace between NaNs, and NaN itself: a write outside it, or a read of a part that was not written, shows
    guard = 1 << 16
    buf = torch.full(((need + 2 * guard) // 4 + 4,), float("nan"), dtype=torch.float32, device="cuda:0").view(torch.uint8)
    B.mc_prefill_attn_paged(dc.params, dc.q, dc.k_pool, dc.v_pool, dc.block_tables, prefix, new, dc.out, dc.lse, buf[guard:guard + need])
    out, lse = dc.result()
    ref_out, ref_lse, _ = oracle.case_full(case)
    check_close(out, ref_out, dtype, "cut")
    assert np.abs(lse - ref_lse).max() <= TOL[dtype]["lse_abs"]
    first = (guard + need + 3) // 4 * 4
    assert torch.isnan(buf[:guard].view(torch.float32)).all() and torch.isnan(buf[first:first + guard].view(torch.float32)).all()
