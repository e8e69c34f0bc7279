"""GPU parity of whole-row attention that is two launches, requests of few rows by the narrow form and the others behind it
(plan_apart in csrc/host_plan.cpp), against the oracle: each dtype, each form of the second launch, requests without new tokens, the few
first or last in the batch; the same bits however the call is driven.  The pools hold NaN behind every request's last key."""
import numpy as np
import pytest
import torch

from paper_2407_00079_amd import binding as B
from paper_2407_00079_amd import workloads as W

from gpu_util import TOL, DeviceCase, check_close

pytestmark = pytest.mark.gpu

APART = 0x4d44                                    # upper half of mc_attn_plan.reserved of such a list

# Hq, Hkv, D, dtype, prefix, new
CASES = [(64, 8, 128, W.BF16, [6000, 0], [3, 900]), (64, 8, 128, W.BF16, [0, 7001], [1100, 33]), (64, 8, 128, W.BF16, [9000, 30], [1, 2200]),
         (64, 8, 128, W.BF16, [17, 5, 12000, 3], [900, 0, 3, 5]), (64, 8, 64, W.BF16, [6000, 0], [3, 900]),
         (64, 8, 64, W.BF16, [12007, 17, 0, 3], [17, 600, 0, 5]), (64, 8, 64, W.BF16, [9000, 30], [1, 2200]),
         (16, 2, 128, W.BF16, [108, 14659, 1947], [2942, 299, 183]),
         (16, 16, 64, W.F32, [3900, 0, 40], [3, 900, 5]), (64, 8, 64, W.F32, [40, 3901, 0], [5, 33, 1100])]


@pytest.mark.parametrize("Hq,Hkv,D,dtype,prefix,new", CASES)
def test_two_launches_match_oracle(oracle, Hq, Hkv, D, dtype, prefix, new):
    print(f"apart case Hq={Hq} Hkv={Hkv} D={D} dtype={dtype} prefix={prefix} new={new}", flush=True)
    pages = sum(-(-(p + c) // 16) for p, c in zip(prefix, new)) + 5
    dc = DeviceCase(W.make_attn_case(99, dtype, Hq, Hkv, D, 16, prefix, new, pages))
    plan_ws = torch.empty_like(dc.workspace)
    plan = B.mc_prefill_attn_prepare(dc.params, prefix, new, 0, plan_ws)
    assert plan.reserved >> 16 == APART
    args = (dc.q, dc.k_pool, dc.v_pool, dc.block_tables)
    ref_out, ref_lse, _ = oracle.case_full(dc.case)
    first = None
    for call in (lambda: B.mc_prefill_attn_run(dc.params, plan, *args, dc.out, dc.lse, plan_ws), dc.run,
                 lambda: B.mc_prefill_attn_paged_noalloc(dc.params, *args, prefix, new, dc.out, dc.lse)):
        dc.out.fill_(float("nan"))
        dc.lse.fill_(float("nan"))
        call()
        out, lse = dc.result()
        check_close(out, ref_out, dtype, "apart")
        assert np.abs(lse - ref_lse).max() <= TOL[dtype]["lse_abs"]
        bits = dc.out.clone(), dc.lse.clone()
        first = first or bits
        assert torch.equal(bits[0], first[0]) and torch.equal(bits[1], first[1])
