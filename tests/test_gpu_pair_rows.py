"""GPU parity of attention by 64-row workgroups whose computing waves are two pairs, each for half of a tile's keys (kPairRows in
csrc/attn_prefill_bf16.hip), against the oracle: ends of rows, of keys and of tiles, requests of one to eight tiles beside a long
one, hard values; whole rows are the same bits however the call is driven.  The pools hold NaN behind every request's last key."""
import numpy as np
import pytest
import torch

from paper_2407_00079_amd import binding as B
from paper_2407_00079_amd import workloads as W

from gpu_util import TOL, DeviceCase, check_close
from test_gpu_nonfinite import poison

pytestmark = pytest.mark.gpu

PAIRS = 0x4d434636                                # mc_attn_plan.reserved of a list that is launched so

# Hq, Hkv, D, prefix, new.  64/8 heads: 130 tokens are 16 row tiles and 16 rows (the second row wave has none), 132 end with 32 rows,
# 133 with 40; 2690 keys end two keys into a tile (the second pair sees none of it), 2688 with one, 2720 and 2721 beside its middle
CASES = [(64, 8, D, [p], [c]) for D in (128, 64) for p, c in ((2560, 130), (2558, 130), (2590, 130), (2591, 130), (2620, 132), (2620, 133))]
CASES += [(12, 3, 128, [2700], [700]), (12, 3, 64, [2700], [700]), (16, 2, 128, [2540], [520]), (16, 16, 128, [2570, 0], [543, 3])]
CASES += [(64, 8, D, [2600, 0, 20, 60, 100, 150, 250, 300, 370], [130, 1, 3, 10, 33, 20, 9, 70, 1]) for D in (128, 64)]
CASES += [(8, 2, D, [2703, 40], [1100, 7]) for D in (128, 64)]


def prepared(Hq, Hkv, D, prefix, new, q_scale=1.0):
    print(f"pairs case Hq={Hq} Hkv={Hkv} D={D} prefix={prefix} new={new} q_scale={q_scale}", flush=True)
    pages = sum(-(-(p + c) // 16) for p, c in zip(prefix, new)) + 5
    dc = DeviceCase(W.make_attn_case(98, W.BF16, Hq, Hkv, D, 16, prefix, new, pages, q_scale=q_scale))
    plan_ws = torch.empty_like(dc.workspace)
    plan = B.mc_prefill_attn_prepare(dc.params, prefix, new, 0, plan_ws)
    assert plan.reserved == PAIRS
    args = (dc.q, dc.k_pool, dc.v_pool, dc.block_tables)
    return dc, (lambda: B.mc_prefill_attn_run(dc.params, plan, *args, dc.out, dc.lse, plan_ws), dc.run,
                lambda: B.mc_prefill_attn_paged_noalloc(dc.params, *args, prefix, new, dc.out, dc.lse))


@pytest.mark.parametrize("Hq,Hkv,D,prefix,new,q_scale", [(*c, 1.0) for c in CASES] + [(*CASES[i], 8.0) for i in (0, 9, 12, 17)])
def test_pair_rows_match_oracle(oracle, Hq, Hkv, D, prefix, new, q_scale):      # 8: references that are raised many times
    dc, calls = prepared(Hq, Hkv, D, prefix, new, q_scale)
    ref_out, ref_lse, _ = oracle.case_full(dc.case)
    first = None
    for call in calls:
        dc.out.fill_(float("nan"))
        dc.lse.fill_(float("nan"))
        call()
        out, lse = dc.result()
        check_close(out, ref_out, W.BF16, "pairs")
        assert np.abs(lse - ref_lse).max() <= TOL[W.BF16]["lse_abs"]
        bits = dc.out.clone(), dc.lse.clone()
        first = first or bits
        assert torch.equal(bits[0], first[0]) and torch.equal(bits[1], first[1])


@pytest.mark.parametrize("what", ["q", "k", "k inf", "new key", "v"])
@pytest.mark.parametrize("D", [128, 64])
def test_pair_rows_are_nan_where_others_are(D, what):
    """A value that is not finite reaches the rows that it reaches by 128-row workgroups (key slices), and no others."""
    dc, calls = prepared(16, 2, D, [2640], [560])
    poison(dc, what)
    calls[2]()
    out, lse = dc.result()
    c, splits, lens = dc.case, 3, ([2640], [560])
    ws = torch.empty(B.mc_prefill_attn_split_workspace_bytes(dc.params, 1, c.total_new, splits), dtype=torch.uint8, device="cuda:0")
    o = torch.empty((splits, c.total_new, 16, D), dtype=torch.float32, device="cuda:0")
    l = torch.empty((splits, c.total_new, 16), dtype=torch.float32, device="cuda:0")
    B.mc_prefill_attn_paged_split(dc.params, dc.q, dc.k_pool, dc.v_pool, dc.block_tables, *lens, splits, o, l, ws)
    B.mc_attn_merge_lse(o, l, splits, c.total_new * 16, D, int(dc.params.dtype), dc.out, dc.lse)
    want, want_lse = dc.result()
    bad = np.isnan(want)
    assert bad.any() and not bad.all()
    assert np.array_equal(np.isnan(out), bad) and np.array_equal(np.isnan(lse), np.isnan(want_lse))
    check_close(out[~bad], want[~bad], W.BF16, "pairs beside slices")
