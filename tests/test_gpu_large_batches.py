"""GPU parity of attention calls of more requests than the kernel argument describes (64 and more with new tokens): lists
uploaded to the workspace, uniform key slices + merge, and the list built on the device in the library's fixed array; and of
63, the most that travel as an argument."""
import numpy as np
import pytest
import torch

from paper_2407_00079_amd import binding as B
from paper_2407_00079_amd import workloads as W

from gpu_util import TOL, DeviceCase, check_close

pytestmark = pytest.mark.gpu


def lengths(requests, most_prefix, most_new, empty_every=0, long=None):
    """Lengths of `requests` requests with new tokens; every empty_every-th place holds one without."""
    rng = np.random.default_rng(requests * 1000 + most_prefix + most_new)
    prefix, new = [], []
    while sum(c > 0 for c in new) < requests:
        none = empty_every and len(new) % empty_every == 0
        prefix.append(int(rng.integers(0, most_prefix + 1)))
        new.append(0 if none else int(rng.integers(1, most_new + 1)))
    if long:
        new[-1] = long
    return prefix, new


# name: dtype, Hq, Hkv, D, (prefix, new)
CASES = {
    "few": (W.BF16, 8, 1, 128, lengths(64, 90, 16)),                            # every row tile of at most 128 rows
    "few, slices": (W.BF16, 8, 1, 128, lengths(66, 1400, 3, empty_every=9)),    # prefixes that pay for key slices
    "halves": (W.BF16, 8, 1, 128, lengths(70, 150, 30, empty_every=5)),         # 70 items: two workgroups each
    "full": (W.BF16, 16, 2, 128, lengths(100, 60, 20, long=70)),                # 202 items and more
    "most requests": (W.BF16, 4, 4, 64, lengths(128, 40, 9)),                   # as many as the fixed array has room for
    "half of them empty": (W.BF16, 4, 1, 64, lengths(64, 70, 40, empty_every=2)),
    "fp32": (W.F32, 4, 1, 64, lengths(80, 100, 40, empty_every=7)),
    "fp32, few": (W.F32, 8, 2, 64, lengths(65, 200, 8)),
    "63": (W.BF16, 16, 2, 128, lengths(63, 300, 25, empty_every=6)),            # the most an argument holds
    "63, fp32": (W.F32, 4, 1, 64, lengths(63, 150, 50)),
}


def make(name, seed=91):
    dtype, Hq, Hkv, D, (prefix, new) = CASES[name]
    pages = sum(-(-(p + c) // 16) for p, c in zip(prefix, new)) + 3
    return DeviceCase(W.make_attn_case(seed, dtype, Hq, Hkv, D, 16, prefix, new, pages)), prefix, new


def noalloc(dc, stream=None):
    B.mc_prefill_attn_paged_noalloc(dc.params, dc.q, dc.k_pool, dc.v_pool, dc.block_tables, dc.case.prefix_lens.tolist(),
                                    dc.case.new_lens.tolist(), dc.out, dc.lse, stream)


def fresh(dc, call):
    dc.out.fill_(float("nan"))
    dc.lse.fill_(float("nan"))
    call()
    torch.cuda.synchronize()
    return dc.out.clone(), dc.lse.clone()


def check(dc, got, ref, what):
    out, lse = got
    check_close(out.float().cpu().numpy().astype(np.float64), ref[0], dc.case.dtype, what)
    assert np.abs(lse.cpu().numpy().astype(np.float64) - ref[1]).max() <= TOL[dc.case.dtype]["lse_abs"], what


@pytest.mark.parametrize("name", CASES)
def test_every_form_matches_oracle(oracle, name):
    print(f"large batch case {name}", flush=True)
    dc, prefix, new = make(name)
    args = (dc.params, dc.q, dc.k_pool, dc.v_pool, dc.block_tables, prefix, new)
    ref = oracle.case_full(dc.case)
    whole = fresh(dc, dc.run)                                    # minimal workspace
    check(dc, whole, ref, "whole rows")
    from_array = fresh(dc, lambda: noalloc(dc))
    assert torch.equal(from_array[0], whole[0]) and torch.equal(from_array[1], whole[1])
    plan_ws = torch.empty_like(dc.workspace)
    plan = B.mc_prefill_attn_prepare(dc.params, prefix, new, 0, plan_ws)
    planned = fresh(dc, lambda: B.mc_prefill_attn_run(dc.params, plan, *args[1:5], dc.out, dc.lse, plan_ws))
    assert torch.equal(planned[0], whole[0]) and torch.equal(planned[1], whole[1])
    need = B.mc_prefill_attn_auto_workspace_bytes(dc.params, prefix, new)
    if name == "few, slices":
        assert B.mc_prefill_attn_suggest_kv_splits(dc.params, prefix, new) > 1
    guard = 1 << 14
    buf = torch.full((need // 4 + 2 * guard,), float("nan"), dtype=torch.float32, device="cuda:0")
    ws = buf[guard:].view(torch.uint8)[:need]
    for call in (B.mc_prefill_attn_paged, B.mc_prefill_attn_auto):
        check(dc, fresh(dc, lambda: call(*args, dc.out, dc.lse, ws)), ref, call.__name__)
    assert torch.isnan(buf[:guard]).all() and torch.isnan(buf[guard + need // 4 + 1:]).all()


def test_a_smaller_batch_after_a_larger_one_runs_only_its_own_items(oracle):
    """Both lists lie in the same array: what the larger one left behind the smaller one must not run."""
    for name in ("most requests", "full", "few", "halves", "few"):
        dc, _, _ = make(name, seed=92)
        check(dc, fresh(dc, lambda: noalloc(dc)), oracle.case_full(dc.case), name)


def test_call_replays_from_a_hip_graph(oracle):
    """Captured once; between the replays, new queries and eager calls that fill the array with other lists."""
    dc, _, _ = make("halves", seed=93)
    other, _, _ = make("full", seed=94)
    noalloc(other)                                               # outside the capture
    side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        noalloc(dc, side)
        side.synchronize()
        with torch.cuda.graph(graph, stream=side):
            noalloc(dc, side)
    torch.cuda.synchronize()
    q = dc.q.clone()
    for turn in range(4):
        dc.q.copy_(q.view(torch.bfloat16).roll(turn, 0).view(torch.int16))
        want = fresh(dc, lambda: noalloc(dc))
        noalloc(other)
        torch.cuda.synchronize()
        got = fresh(dc, graph.replay)
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1]), turn
        assert torch.isfinite(got[1]).all()
