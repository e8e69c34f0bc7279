"""GPU parity of the calls whose request and offset tables travel in the kernel argument up to 64 entries and are uploaded
beyond: append, prefix keys and prefix match on both sides of that line, byte for byte against the CPU oracle."""
import numpy as np
import pytest
import torch

from paper_2407_00079_amd import binding as B
from paper_2407_00079_amd import workloads as W

from append_util import empty_chunk_pools, new_rows
from gpu_util import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("batch", [1, 63, 64, 65])
@pytest.mark.parametrize("dtype,D,Hkv", [(W.BF16, 128, 1), (W.BF16, 64, 3)])
def test_append(oracle, batch, dtype, D, Hkv):
    print(f"append tables batch={batch} D={D} Hkv={Hkv}", flush=True)
    # one-token requests (a wave spans several), runs of empty ones at the front, inside and at the end
    new = [(0, 1, 0, 7, 1, 1, 30, 0)[r % 8] for r in range(batch)]
    new[batch // 2] += 1
    prefix = [(3 * r) % 50 for r in range(batch)]
    case = W.make_attn_case(31, dtype, 2 * Hkv, Hkv, D, 16, prefix, new, 6 * batch + 8, keep_logical=True)
    k0, v0 = empty_chunk_pools(case)
    k_new, v_new = new_rows(case)
    k_dev, v_dev = dev(k0), dev(v0)
    params = B.attn_params(case.num_q_heads, Hkv, D, 16, case.num_pages, dtype)
    ws = torch.empty(B.mc_kv_append_workspace_bytes(batch), dtype=torch.uint8, device="cuda:0")
    B.mc_kv_append_paged(params, dev(k_new), dev(v_new), k_dev, v_dev, dev(case.block_tables), prefix, new, ws)
    torch.cuda.synchronize()
    oracle.kv_append_paged(k_new, v_new, k0, v0, case.block_tables, prefix, new)
    np.testing.assert_array_equal(k_dev.cpu().numpy().view(k0.dtype), k0)
    np.testing.assert_array_equal(v_dev.cpu().numpy().view(v0.dtype), v0)


@pytest.mark.parametrize("batch,n_inst", [(64, 64), (65, 3), (3, 65), (64, 1)])
def test_prefix(oracle, batch, n_inst):
    print(f"prefix tables batch={batch} n_inst={n_inst}", flush=True)
    rng = np.random.default_rng(batch * 100 + n_inst)
    lens = [int(x) for x in rng.integers(0, 700, size=batch)]
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    tokens = rng.integers(-5, 128000, size=int(off[-1]), dtype=np.int32)
    ref, koff = oracle.prefix_hash(tokens, off, 16)
    keys = torch.full((len(ref),), -1, dtype=torch.int64, device="cuda:0")
    ws = torch.empty(B.mc_prefix_hash_workspace_bytes(batch), dtype=torch.uint8, device="cuda:0")
    B.mc_prefix_hash(dev(tokens), off.tolist(), 16, keys, ws)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(keys.cpu().numpy().view(np.uint64), ref)
    cache = []
    for i in range(n_inst):      # a leading part of every request, more of it the later the instance
        held = [ref[koff[r]:koff[r] + (koff[r + 1] - koff[r]) * i // n_inst] for r in range(batch)]
        cache.append(np.unique(np.concatenate(held + [rng.integers(0, 1 << 63, size=i, dtype=np.uint64)])))
    coff = np.concatenate([[0], np.cumsum([c.size for c in cache])]).astype(np.int64)
    ck = np.concatenate(cache).astype(np.uint64)
    want = oracle.prefix_match(ref, koff, ck, coff)
    got = [torch.full((batch, n_inst), -7, dtype=torch.int32, device="cuda:0"),
           torch.full((batch,), -7, dtype=torch.int32, device="cuda:0"), torch.full((batch,), -7, dtype=torch.int32, device="cuda:0")]
    ws = torch.empty(B.mc_prefix_match_workspace_bytes(batch, n_inst), dtype=torch.uint8, device="cuda:0")
    B.mc_prefix_match(keys, koff.tolist(), dev(ck.view(np.int64)), coff.tolist(), *got, ws)
    torch.cuda.synchronize()
    for g, w in zip(got, want):
        np.testing.assert_array_equal(g.cpu().numpy(), w)
