"""GPU parity of the one-shot attention call with room for partial results: row tiles cut into pieces along the keys
(classes in the kernel argument) and their merge, against the oracle, at the edges of row tiles, key tiles and pieces.  All but
two of the shapes (one key; 127, 128 with 1000, 60) take narrow row tiles; the wide ones, cut, are in test_gpu_wide_rows.py and
in the second half of PIECES in test_gpu_narrow.py."""
import numpy as np
import pytest
import torch

from paper_2407_00079_amd import binding as B
from paper_2407_00079_amd import workloads as W

from gpu_util import TOL, DeviceCase, check_close

pytestmark = pytest.mark.gpu

# dtype, Hq, Hkv, D, prefix, new
CASES = [
    (W.F32, 4, 1, 64, [256], [128]),                          # row tiles of six key tiles and less
    (W.F32, 4, 4, 64, [0, 65], [257, 1]),                     # no prefix; a row tile of one row; one key tile and a key
    (W.BF16, 8, 1, 128, [0], [1]),                            # one row, one key
    (W.BF16, 64, 8, 128, [1023, 64], [1, 33]),                # a tile of 8 rows; 33 tokens: 264 rows, the last tile of 8
    (W.BF16, 8, 2, 128, [919], [355]),                        # early row tiles see fewer key tiles than there are pieces
    (W.BF16, 16, 16, 128, [538, 0, 7], [94, 0, 300]),         # one head per group, an empty request, row tiles at 256 rows
    (W.BF16, 12, 3, 128, [2000, 3], [40, 86]),                # groups of 4 heads, three KV heads
    (W.BF16, 16, 2, 64, [1500, 31], [17, 129]),               # 128-byte rows
    (W.BF16, 64, 8, 128, [127, 128], [1000, 60]),             # one full round of row tiles and a rest that is cut
    (W.BF16, 8, 1, 128, [40000], [9]),                        # 72 rows; pieces of several key tiles
    (W.BF16, 16, 1, 128, [9000, 63, 320], [8, 1, 5]),         # 128, 16 and 80 rows
    (W.BF16, 64, 8, 64, [9999], [17]),                        # 136 rows: the last row tile of 8
    (W.F32, 8, 2, 64, [3000], [33]),
]


@pytest.mark.parametrize("dtype,Hq,Hkv,D,prefix,new", CASES)
def test_pieces_match_oracle(oracle, dtype, Hq, Hkv, D, prefix, new):
    print(f"pieces case {dtype} Hq={Hq} Hkv={Hkv} D={D} prefix={prefix} new={new}", flush=True)
    pages = sum(-(-(p + c) // 16) for p, c in zip(prefix, new)) + 5
    case = W.make_attn_case(71, dtype, Hq, Hkv, D, 16, prefix, new, pages)
    dc = DeviceCase(case)
    need = B.mc_prefill_attn_auto_workspace_bytes(dc.params, prefix, new)
    # the partial results lie between NaNs: a write outside them, or a read of a part that was not written, shows
    guard = 1 << 16
    buf = torch.full(((need + 2 * guard) // 4 + 4,), float("nan"), dtype=torch.float32, device="cuda:0").view(torch.uint8)
    ws = buf[guard:guard + need]
    B.mc_prefill_attn_paged(dc.params, dc.q, dc.k_pool, dc.v_pool, dc.block_tables, prefix, new, dc.out, dc.lse, ws)
    out, lse = dc.result()
    ref_out, ref_lse, _ = oracle.case_full(case)
    check_close(out, ref_out, dtype, "pieces")
    assert np.abs(lse - ref_lse).max() <= TOL[dtype]["lse_abs"]
    first = (guard + need + 3) // 4 * 4
    assert torch.isnan(buf[:guard].view(torch.float32)).all() and torch.isnan(buf[first:first + guard].view(torch.float32)).all()


@pytest.mark.parametrize("dtype,D,tiles", [(W.BF16, 128, n) for n in (1, 2, 3, 4, 5, 6, 7, 11)] + [(W.BF16, 64, 6), (W.F32, 64, 5)])
def test_few_rows_without_room(oracle, dtype, D, tiles):
    """No room for partial results: a workgroup walks all key tiles of its rows, one tile and up to eleven (narrow row tiles but for
    one key tile; the key slices below take 128-row ones, over as many tiles as there are LDS buffers and around that); rows for
    one row tile and for several."""
    for new in (1, 7, 16, 33):                                # 33 tokens: the last row tile of 8 rows
        print(f"few rows case {dtype} D={D} tiles={tiles} new={new}", flush=True)
        case = W.make_attn_case(72 + tiles, dtype, 16, 2, D, 16, [64 * tiles - new - 3], [new], 4 * tiles + 3)
        dc = DeviceCase(case)
        dc.run()
        out, lse = dc.result()
        ref_out, ref_lse, _ = oracle.case_full(case)
        check_close(out, ref_out, dtype, "few rows")
        assert np.abs(lse - ref_lse).max() <= TOL[dtype]["lse_abs"]
        # the same from a prepared list, whole rows and key slices (some of them without a key a row may see)
        p, args = dc.params, (dc.q, dc.k_pool, dc.v_pool, dc.block_tables)
        dc.out.fill_(float("nan"))
        dc.lse.fill_(float("nan"))
        plan = B.mc_prefill_attn_prepare(p, case.prefix_lens.tolist(), case.new_lens.tolist(), 0, dc.workspace)
        B.mc_prefill_attn_run(p, plan, *args, dc.out, dc.lse, dc.workspace)
        check_close(dc.result()[0], ref_out, dtype, "few rows, planned")
        ws = torch.empty(B.mc_prefill_attn_split_workspace_bytes(p, 1, new, 3), dtype=torch.uint8, device="cuda:0")
        o_parts = torch.full((3, new, 16, D), float("nan"), dtype=torch.float32, device="cuda:0")
        lse_parts = torch.full((3, new, 16), float("nan"), dtype=torch.float32, device="cuda:0")
        plan = B.mc_prefill_attn_prepare(p, case.prefix_lens.tolist(), case.new_lens.tolist(), 3, ws)
        B.mc_prefill_attn_run_split(p, plan, *args, o_parts, lse_parts, ws)
        dc.out.fill_(float("nan"))
        B.mc_attn_merge_lse(o_parts, lse_parts, 3, new * 16, D, int(p.dtype), dc.out, dc.lse)
        out, lse = dc.result()
        check_close(out, ref_out, dtype, "few rows, split")
        assert np.abs(lse - ref_lse).max() <= TOL[dtype]["lse_abs"]
