"""GPU parity of the attention kernels of 128- and 256-row workgroups where small shapes run the narrow form: hard values, the
softmax reference, NaN, prepared plans and graphs.  Every test says which form its lengths take."""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2407_00079_amd import binding as B
from paper_2407_00079_amd import workloads as W

from append_util import empty_chunk_pools, new_rows
from gpu_util import TOL, DeviceCase, check_close, dev
from test_gpu_nonfinite import pieces, poison, whole
from test_gpu_random import random_shape
from wide_util import CUT, HEADS, WHOLE, rows_of_list, with_short_requests

pytestmark = pytest.mark.gpu


def device_case(case, rows=None):
    dc = DeviceCase(case)
    got = rows_of_list(dc.params, case.prefix_lens.tolist(), case.new_lens.tolist(), torch.empty_like(dc.workspace))
    print(f"wide case {case.dtype} rows={got} Hq={case.num_q_heads} Hkv={case.num_kv_heads} D={case.head_dim} "
          f"prefix={case.prefix_lens.tolist()[:4]} new={case.new_lens.tolist()[:4]} seed={case.seed}", flush=True)
    assert rows in (None, got)
    return dc


def make(seed, dtype, D, prefix, new, **kw):
    pages = sum(-(-(p + c) // 16) for p, c in zip(prefix, new)) + 5
    return W.make_attn_case(seed, dtype, *HEADS, D, 16, prefix, new, kw.pop("pages", pages), **kw)


def check(oracle, dc, call, scale=0.0, what=""):
    dc.out.fill_(float("nan"))
    dc.lse.fill_(float("nan"))
    call()
    out, lse = dc.result()
    ref_out, ref_lse, _ = oracle.case_full(dc.case, scale or None)
    check_close(out, ref_out, dc.case.dtype, what)
    assert np.abs(lse - ref_lse).max() <= TOL[dc.case.dtype]["lse_abs"], what
    return dc.out.clone(), dc.lse.clone()


def same(a, b):
    return all(torch.equal(x, y) for x, y in zip(a, b))


@pytest.mark.parametrize("rows,dtype,D,prefix,new", WHOLE)
def test_large_scores_scale_paging_and_poison(oracle, rows, dtype, D, prefix, new):
    """Scores of tens of units (fp32: what its tolerance bears) and a scale of the caller's own, against the oracle; the same bits
    without lse, from other pages, and whatever lies behind the last key."""
    case = make(81, dtype, D, prefix, new, q_scale=30.0 if dtype == W.BF16 else 8.0, keep_logical=True)
    dc = device_case(case, rows)
    check(oracle, dc, dc.run, what="large scores")
    got = check(oracle, dc, lambda: dc.run(0.02), 0.02, "scale 0.02")
    dc.out.fill_(float("nan"))
    dc.lse.fill_(7.0)
    dc.run(0.02, want_lse=False)
    torch.cuda.synchronize()
    assert torch.equal(dc.out, got[0]) and (dc.lse == 7.0).all()
    logical = (case.q, case.k_logical, case.v_logical)
    for other in (make(82, dtype, D, prefix, new, logical=logical, pages=777), make(81, dtype, D, prefix, new, logical=logical, poison=False)):
        oc = device_case(other, rows)
        oc.run(0.02)
        torch.cuda.synchronize()
        assert same((oc.out, oc.lse), got)


@pytest.mark.parametrize("rows,D,prefix,new", [(rows, D, prefix, new) for rows, dtype, D, prefix, new in WHOLE if dtype == W.BF16])
def test_scores_that_keep_outgrowing_the_reference(oracle, rows, D, prefix, new):
    """Scores that rise along the keys at eight different rates, one per head of a group (from 0.3 to 20 log2 units per 32-key
    block): the lazy softmax reference is outgrown by just under and just over its margin again and again, in the pipelined
    tiles (the prefix) and in the diagonal ones."""
    (Hq, Hkv), (P,), (C,) = HEADS, prefix, new
    rng = np.random.default_rng(11)
    u = rng.standard_normal(D)
    u /= np.linalg.norm(u)
    rates = np.tile([0.3, 3.0, 6.9, 7.4, 7.9, 8.1, 12.0, 20.0], Hkv)            # log2 units per 32 keys
    ramp = (np.arange(P + C) / 32.0)[:, None, None]
    k = (ramp * u + 0.05 * rng.standard_normal((P + C, Hkv, D))).astype(np.float32)
    v = rng.standard_normal((P + C, Hkv, D)).astype(np.float32)
    q = (rates[:, None] * np.sqrt(D) / np.log2(np.e) * u + 0.05 * rng.standard_normal((C, Hq, D))).astype(np.float32)
    bits = W.f32_to_bf16_bits
    dc = device_case(make(12, W.BF16, D, prefix, new, logical=(bits(q), [bits(k)], [bits(v)])), rows)
    check(oracle, dc, dc.run, what="rising scores")


@pytest.mark.parametrize("rows,C", [(128, 130), (256, 600)])
def test_needle_through_block_table(oracle, rows, C):
    """A key aligned with one row of Q dominates it: its output is that key's V row."""
    (Hq, Hkv), D, P = HEADS, 128, 720
    L = P + C
    rng = np.random.default_rng(3)
    q = rng.standard_normal((C, Hq, D)).astype(np.float32)
    v = rng.standard_normal((L, Hkv, D)).astype(np.float32)
    k = (0.01 * rng.standard_normal((L, Hkv, D))).astype(np.float32)
    needles = dict(zip(range(0, Hq, Hq // Hkv), (0, 15, 16, 719, 720, 777, L - 2, L - 1)))   # one a KV head
    for head, needle in needles.items():
        k[needle, head * Hkv // Hq] = 60.0 * q[C - 1, head] / np.linalg.norm(q[C - 1, head])
    bits = W.f32_to_bf16_bits
    dc = device_case(make(7, W.BF16, D, [P], [C], logical=(bits(q), [bits(k)], [bits(v)])), rows)
    check(oracle, dc, dc.run, what="needles")
    out = dc.result()[0]
    for head, needle in needles.items():
        row = W.bf16_bits_to_f32(bits(v[needle, head * Hkv // Hq])).astype(np.float64)
        assert np.abs(out[C - 1, head] - row).max() <= 2e-2


@pytest.mark.parametrize("rows,new", [(128, [210, 150]), (256, [500, 350])])
def test_shared_prefix_pages(oracle, rows, new):
    dc = device_case(make(5, W.BF16, 128, [768, 768], new, shared_prefix_pages=48), rows)
    check(oracle, dc, dc.run, what="shared prefix")


def test_chunked_calls_match_one_call(oracle):
    """One call of 256-row workgroups, its two chunks of 128-row ones."""
    case = make(41, W.BF16, 128, [128], [700])
    one = device_case(case, 256)
    at_once = check(oracle, one, one.run, what="one call")[0].float()
    c1, parts = 300, []
    for q, p, c in ((case.q[:c1], 128, c1), (case.q[c1:], 128 + c1, 700 - c1)):
        dc = device_case(dataclasses.replace(case, q=q, prefix_lens=np.array([p], np.int32), new_lens=np.array([c], np.int32)), 128)
        parts.append(check(oracle, dc, dc.run, what=f"chunk behind {p}")[0].float())
    assert (torch.cat(parts) - at_once).abs().max() <= 2e-2


@pytest.mark.parametrize("what", ["q", "k", "k inf", "new key", "v"])
@pytest.mark.parametrize("rows,dtype,D,prefix,new", CUT)
def test_cut_rows_are_nan_where_whole_rows_are(rows, dtype, D, prefix, new, what):
    dc = device_case(make(83, dtype, D, prefix, new))
    poison(dc, what)
    whole(dc)
    want_o, want_l = dc.result()
    bad = np.isnan(want_o)
    assert bad.any() and not bad.all()
    dc.out.fill_(7.0)
    dc.lse.fill_(7.0)
    pieces(dc)
    got_o, got_l = dc.result()
    np.testing.assert_array_equal(np.isnan(got_o), bad)
    np.testing.assert_array_equal(np.isnan(got_l), np.isnan(want_l))
    assert not np.isinf(got_l).any()
    assert np.abs(got_o[~bad] - want_o[~bad]).max() <= 2 * TOL[dtype]["max_abs"]     # two roundings of the same rows


@pytest.mark.parametrize("rows,dtype,D,prefix,new", CUT)
def test_cut_rows_match_oracle(oracle, rows, dtype, D, prefix, new):
    dc = device_case(make(84, dtype, D, prefix, new, q_scale=4.0))
    check(oracle, dc, lambda: pieces(dc), what="cut")


@pytest.mark.parametrize("rows,prefix,new", [(128, [700, 0, 33], [300, 129, 1]), (256, [700, 0, 33], [600, 429, 1])])
def test_a_plan_and_its_graph_give_what_one_call_gives(oracle, rows, prefix, new):
    """append_run + attn_run from a prepared plan, eagerly and from a graph, with other values in eager work between the replays."""
    side, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    case = make(900, W.BF16, 128, prefix, new, keep_logical=True)
    dc = device_case(case, rows)
    k0, v0 = (dev(x) for x in empty_chunk_pools(case))
    dc.k_pool, dc.v_pool = k0.clone(), v0.clone()
    k_new, v_new = (dev(x) for x in new_rows(case))
    ws = torch.empty_like(dc.workspace)

    def step():
        B.mc_kv_append_run(dc.params, plan, k_new, v_new, dc.k_pool, dc.v_pool, dc.block_tables, ws, side)
        B.mc_prefill_attn_run(dc.params, plan, dc.q, dc.k_pool, dc.v_pool, dc.block_tables, dc.out, dc.lse, ws, side)

    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        plan = B.mc_prefill_attn_prepare(dc.params, prefix, new, 0, ws, side)
        step()
        side.synchronize()
        with torch.cuda.graph(graph, stream=side):
            step()
    torch.cuda.synchronize()
    got = [dc.out.clone(), dc.lse.clone()]
    np.testing.assert_array_equal(dc.k_pool.cpu().numpy().view(np.uint16), case.k_pool)
    want = check(oracle, dc, dc.run, what="one call")
    assert same(got, want)
    q = dc.q.clone()
    for turn in range(1, 4):
        dc.q.copy_(q.roll(turn, 0))
        dc.k_pool.copy_(k0)
        dc.v_pool.copy_(v0)
        dc.out.fill_(float("nan"))
        dc.lse.fill_(float("nan"))
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        got = [dc.out.clone(), dc.lse.clone()]
        dc.run()
        torch.cuda.synchronize()
        assert same(got, (dc.out, dc.lse)) and torch.isfinite(got[1]).all(), turn


@pytest.mark.parametrize("dtype,D,tiles", [(W.BF16, 128, n) for n in (1, 2, 3, 4, 5, 6, 7, 11)] + [(W.BF16, 64, 6), (W.F32, 64, 5)])
def test_few_rows_and_as_many_key_tiles_as_there_are_buffers(oracle, dtype, D, tiles):
    """128-row workgroups whose rows fill one, two and four of the computing waves, and two workgroups of an item (33 tokens), over
    as many key tiles as there are LDS buffers and around that; one call and a prepared list."""
    for new in (1, 7, 16, 33):
        prefix, chunks = with_short_requests([64 * tiles - new - 3], [new])
        case = W.make_attn_case(72 + tiles, dtype, 8, 1, D, 16, prefix, chunks, 4 * tiles + 70)
        dc = device_case(case, 128)
        one = check(oracle, dc, dc.run, what="few rows")
        ws = torch.empty_like(dc.workspace)
        plan = B.mc_prefill_attn_prepare(dc.params, prefix, chunks, 0, ws)
        run = lambda: B.mc_prefill_attn_run(dc.params, plan, dc.q, dc.k_pool, dc.v_pool, dc.block_tables, dc.out, dc.lse, ws)
        assert same(check(oracle, dc, run, what="few rows, planned"), one)


@pytest.mark.parametrize("seed", range(24))
def test_random_shapes_match_oracle(oracle, seed):
    """The shapes of test_gpu_random.py, most of which run the narrow form, among so many short requests that they do not."""
    dtype, Hq, Hkv, D, prefix, new, pages, _ = random_shape(seed)
    prefix, new = with_short_requests(prefix, new)
    dc = device_case(W.make_attn_case(2100 + seed, dtype, Hq, Hkv, D, 16, prefix, new, pages + 64, q_scale=4.0))
    check(oracle, dc, dc.run, what="whole rows")
