"""GPU parity of narrow row tiles whose output columns several workgroups share (csrc/attn_narrow.hip), on both sides of every
line of narrow_shares (csrc/host_plan.cpp), against the oracle; a row tile is the same bits however many take it (a prepared list
counts its row tiles roughly, so beside a line the calls take different shares)."""
import numpy as np
import pytest
import torch

from paper_2407_00079_amd import binding as B
from paper_2407_00079_amd import workloads as W

from gpu_util import TOL, DeviceCase, check_close
from test_gpu_narrow import LEAST, NARROW

pytestmark = pytest.mark.gpu

# dtype, Hq, Hkv, D, prefix, new: 48, 49, 96, 97 row tiles of 32 rows (the second and fourth end in one of 8); of 16 rows 48, 64, 96, 112
SHARED = [(W.BF16, 8, 1, D, [701], [new]) for D in (128, 64) for new in (192, 193, 384, 385)]
SHARED += [(W.BF16, 16, 16, D, [333, 64, 500, 95, 31, 257, 640][:n], [16, 1, 7, 16, 16, 9, 2][:n]) for D in (128, 64) for n in (3, 4, 6, 7)]
# fp32: 64, 65, 128, 129
SHARED += [(W.F32, 4, 1, 64, [301], [new]) for new in (256, 257, 512, 513)]


@pytest.mark.parametrize("dtype,Hq,Hkv,D,prefix,new", SHARED)
def test_shares_of_a_row_tile_match_oracle(oracle, dtype, Hq, Hkv, D, prefix, new):
    print(f"shares case {dtype} Hq={Hq} Hkv={Hkv} D={D} prefix={prefix} new={new}", flush=True)
    pages = sum(-(-(p + c) // 16) for p, c in zip(prefix, new)) + 5
    case = W.make_attn_case(97, dtype, Hq, Hkv, D, 16, prefix, new, pages, q_scale=2.0)
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
        check_close(out, ref_out, dtype, "shares")
        assert np.abs(lse - ref_lse).max() <= TOL[dtype]["lse_abs"]
        bits = dc.out.clone(), dc.lse.clone()
        first = first or bits
        assert torch.equal(bits[0], first[0]) and torch.equal(bits[1], first[1])
