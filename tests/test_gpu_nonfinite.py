"""GPU: a NaN or an infinity in Q or in a visible K or V row reaches the output of row tiles cut into pieces or slices just
as it reaches whole rows, and rows that do not see it stay what they are."""
import numpy as np
import pytest
import torch

from paper_2407_00079_amd import binding as B
from paper_2407_00079_amd import workloads as W

from gpu_util import TOL, DeviceCase, dev

pytestmark = pytest.mark.gpu

# dtype, Hq, Hkv, D, prefix, new: all of them in the narrow form, the second, third and fifth cut into pieces where the workspace
# has room (against whole narrow row tiles), and all against key slices of 128- and 256-row tiles; cut wide row tiles are in
# test_gpu_wide_rows.py
SHAPES = [(W.F32, 4, 1, 64, [256], [128]), (W.BF16, 64, 8, 128, [4000], [16]), (W.BF16, 16, 2, 64, [3000], [40]),
          (W.BF16, 8, 2, 128, [700, 1500], [90, 3]), (W.F32, 8, 2, 64, [3000, 5], [33, 2])]


def poison(dc, what):
    """One non-finite value in a place that some rows of the first request see and rows of other heads do not."""
    nan, inf = float("nan"), float("inf")
    view = (lambda t: t.view(torch.bfloat16)) if dc.case.dtype == W.BF16 else (lambda t: t)
    page = int(dc.case.block_tables[0, 3])
    if what == "q":
        view(dc.q)[2, 1, 3] = nan
    elif what == "new key":                       # the key of the chunk's last token: only that token's rows see it
        pos = int(dc.case.prefix_lens[0] + dc.case.new_lens[0]) - 1
        view(dc.k_pool)[int(dc.case.block_tables[0, pos // 16]), 0, pos % 16, 7] = nan
    else:
        pool = dc.v_pool if what == "v" else dc.k_pool
        view(pool)[page, 0, 5, 7] = inf if what == "k inf" else nan


def whole(dc):
    B.mc_prefill_attn_paged_noalloc(dc.params, dc.q, dc.k_pool, dc.v_pool, dc.block_tables, dc.case.prefix_lens.tolist(),
                                    dc.case.new_lens.tolist(), dc.out, dc.lse)


def pieces(dc):
    lens = dc.case.prefix_lens.tolist(), dc.case.new_lens.tolist()
    need = B.mc_prefill_attn_auto_workspace_bytes(dc.params, *lens)
    assert need > B.mc_prefill_attn_workspace_bytes(dc.params, dc.case.batch, dc.case.total_new)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda:0")
    B.mc_prefill_attn_paged(dc.params, dc.q, dc.k_pool, dc.v_pool, dc.block_tables, *lens, dc.out, dc.lse, ws)


def slices(splits):
    def run(dc):
        c, lens = dc.case, (dc.case.prefix_lens.tolist(), dc.case.new_lens.tolist())
        ws = torch.empty(B.mc_prefill_attn_split_workspace_bytes(dc.params, c.batch, c.total_new, splits), dtype=torch.uint8, device="cuda:0")
        o = torch.full((splits, c.total_new, c.num_q_heads, c.head_dim), float("nan"), dtype=torch.float32, device="cuda:0")
        l = torch.full((splits, c.total_new, c.num_q_heads), float("nan"), dtype=torch.float32, device="cuda:0")
        B.mc_prefill_attn_paged_split(dc.params, dc.q, dc.k_pool, dc.v_pool, dc.block_tables, *lens, splits, o, l, ws)
        B.mc_attn_merge_lse(o, l, splits, c.total_new * c.num_q_heads, c.head_dim, int(dc.params.dtype), dc.out, dc.lse)
    return run


@pytest.mark.parametrize("what", ["q", "k", "k inf", "new key", "v"])
@pytest.mark.parametrize("dtype,Hq,Hkv,D,prefix,new", SHAPES)
def test_cut_rows_are_nan_where_whole_rows_are(dtype, Hq, Hkv, D, prefix, new, what):
    print(f"non-finite case {what}: {dtype} Hq={Hq} Hkv={Hkv} D={D} prefix={prefix} new={new}", flush=True)
    pages = sum(-(-(p + c) // 16) for p, c in zip(prefix, new)) + 5
    dc = DeviceCase(W.make_attn_case(81, dtype, Hq, Hkv, D, 16, prefix, new, pages))
    poison(dc, what)
    whole(dc)
    want_o, want_l = dc.result()
    bad = np.isnan(want_o)
    assert bad.any()
    for form in (pieces, slices(3), slices(11)):
        dc.out.fill_(7.0)
        dc.lse.fill_(7.0)
        form(dc)
        got_o, got_l = dc.result()
        np.testing.assert_array_equal(np.isnan(got_o), bad)
        np.testing.assert_array_equal(np.isnan(got_l), np.isnan(want_l))
        assert not np.isinf(got_l).any()
        # two roundings of the same rows
        assert np.abs(got_o[~bad] - want_o[~bad]).max(initial=0.0) <= 2 * TOL[dtype]["max_abs"]


@pytest.mark.parametrize("parts", [3, 7, 8, 40])
@pytest.mark.parametrize("dtype,D", [(W.BF16, 128), (W.BF16, 64), (W.F32, 64)])
def test_merge_leaves_out_parts_without_keys_and_nothing_else(oracle, parts, dtype, D):
    """Rows of foreign partials with a NaN log-sum-exp, a NaN or an infinite column in a part of any weight, before and behind
    the heaviest part; parts without keys whose columns hold NaN."""
    print(f"merge case parts={parts} {dtype} D={D}", flush=True)
    rng = np.random.default_rng(parts)
    rows = 4 * parts + 3
    o = rng.standard_normal((parts, rows, D)).astype(np.float32)
    l = (3 * rng.standard_normal((parts, rows))).astype(np.float32)
    for s in range(parts):
        l[s, s] = np.nan
        o[s, parts + s, 3] = np.inf
        l[s, parts + s] -= 60.0                    # far below the rest, not so far that its weight is 0
        o[s, 2 * parts + s, 5] = np.nan
        l[s, 3 * parts + s] = -np.inf              # no keys
        o[s, 3 * parts + s] = np.nan
    l[:, -1] = -np.inf                             # no part has keys
    l[:, -2] = -np.inf                             # one part is NaN, the others have no keys
    l[parts - 1, -2] = np.nan
    out = torch.full((rows, D), 7.0, dtype=torch.bfloat16 if dtype == W.BF16 else torch.float32, device="cuda:0")
    lse = torch.full((rows,), 7.0, dtype=torch.float32, device="cuda:0")
    B.mc_attn_merge_lse(dev(o), dev(l), parts, rows, D, B.MC_DTYPE_BF16 if dtype == W.BF16 else B.MC_DTYPE_F32, out, lse)
    torch.cuda.synchronize()
    got, got_l = out.float().cpu().numpy().astype(np.float64), lse.cpu().numpy().astype(np.float64)
    with np.errstate(invalid="ignore"):
        want, want_l = oracle.attn_merge_lse(o, l)
    want[-2], want_l[-2] = np.nan, np.nan          # (the oracle's maximum passes a NaN over)
    np.testing.assert_array_equal(np.isnan(got), np.isnan(want))
    np.testing.assert_array_equal(np.isinf(got), np.isinf(want))
    np.testing.assert_array_equal(np.isnan(got_l), np.isnan(want_l))
    assert np.isneginf(got_l[-1]) and (got[-1] == 0).all()
    fine = np.isfinite(want)
    tol = 2.0 ** -8 * max(1.0, np.abs(want[fine]).max()) if dtype == W.BF16 else 1e-5      # one rounding to bf16
    assert np.abs(got[fine] - want[fine]).max() <= tol
    keep = np.isfinite(want_l)
    assert np.abs(got_l[keep] - want_l[keep]).max() <= 1e-5 * np.abs(want_l[keep]).max()
