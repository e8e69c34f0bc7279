"""GPU parity of prefix keys and match at the lines between the kernels that compute them (one launch for requests of few
blocks, digests and chains in stages for long ones; one workgroup per request or per pair), bit for bit against the oracle."""
import numpy as np
import pytest
import torch

from paper_2407_00079_amd import binding as B

from gpu_util import dev
from test_gpu_prefix import gpu_keys

pytestmark = pytest.mark.gpu

BT = 16
# blocks per request (a request has one token less than that many blocks hold, so its last block is partial)
CASES = [
    [1], [15, 16, 17, 0, 3], [32, 4, 31, 5], [33], [33, 0, 1, 32, 4], [2] * 66 + [32],
    [64, 63, 65, 100, 7],
    [96 + r for r in range(64)],                      # first blocks chained beside the digests of the rest
    [0, 400] + [130] * 61 + [1],                      # ... in requests that end before, at and after the line
    [144] * 46 + [143, 145, 16],
    [7001],                                           # one request that long
    [96] * 70,                                        # tables of more than 64 requests, in device memory
]


@pytest.mark.parametrize("blocks", CASES)
def test_keys_match_oracle(oracle, blocks):
    print(f"prefix stages case blocks={blocks[:6]} of {len(blocks)}", flush=True)
    rng = np.random.default_rng(sum(blocks))
    lens = [max(n * BT - 1, 0) for n in blocks]
    tokens = rng.integers(-5, 128000, size=sum(lens), dtype=np.int32)
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    ref, _ = oracle.prefix_hash(tokens, off, BT)
    np.testing.assert_array_equal(gpu_keys(tokens, off, BT), ref)


@pytest.mark.parametrize("block,lens", [
    (640, [20480, 3, 0, 641]), (640, [20480, 20481]),                   # 32 blocks of one launch, and a token too many
    (8192, [4 * 8192, 8192, 1]), (8192, [4 * 8192 + 1]),                # a SIMD for every block, and a block too many
    (4096, [32 * 4096 - 7, 4096]), (1 << 20, [100, 0, 5000]),
])
def test_keys_of_long_blocks_match_oracle(oracle, block, lens):
    print(f"prefix long blocks case block={block} lens={lens}", flush=True)
    tokens = np.random.default_rng(block).integers(-5, 128000, size=sum(lens), dtype=np.int32)
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    ref, _ = oracle.prefix_hash(tokens, off, block)
    np.testing.assert_array_equal(gpu_keys(tokens, off, block), ref)


def _caches(rng):
    top = (1 << 64) - 1
    yield np.zeros(0, dtype=np.uint64)
    yield np.array([0], dtype=np.uint64)
    yield np.array([5, top], dtype=np.uint64)
    yield np.array([0, 0, 7, 7, 7, top, top], dtype=np.uint64)                                    # repeats
    yield np.arange(1, 701, dtype=np.uint64) * np.uint64(3)                                       # spread evenly, far from hashes
    yield np.sort(rng.integers(0, 1 << 64, size=5000, dtype=np.uint64))                           # what hashes look like
    yield np.sort(np.concatenate([rng.integers(0, 1000, size=400, dtype=np.uint64),               # two clusters and a lone key
                                  rng.integers(top - 100000, top, size=900, dtype=np.uint64), np.array([1 << 40], dtype=np.uint64)]))
    yield np.uint64(1) << np.arange(64, dtype=np.uint64)                                          # ever wider gaps
    yield np.sort(np.exp2(rng.uniform(0, 63.9, size=3000)).astype(np.uint64))


@pytest.mark.parametrize("per_request,requests", [(1, 60), (1, 700), (113, 8), (114, 8), (300, 3)])
def test_match_over_any_ascending_keys(oracle, per_request, requests):
    """9 instances: up to 113 keys a request are looked up by one workgroup (1024 pairs), more by one per instance."""
    print(f"prefix match case per_request={per_request} requests={requests}", flush=True)
    rng = np.random.default_rng(per_request + requests)
    caches = list(_caches(rng))
    held = np.concatenate(caches)
    near = np.concatenate([held, held + np.uint64(1), held - np.uint64(1), rng.integers(0, 1 << 64, size=50, dtype=np.uint64)])
    keys = []
    for r in range(requests):         # keys an instance holds (so that a match gets past the first), then any
        own = caches[r % len(caches)]
        k = rng.choice(own, size=per_request) if len(own) else np.zeros(per_request, dtype=np.uint64)
        k[int(rng.integers(0, per_request + 1)):] = rng.choice(near)
        keys.append(rng.choice(near, size=per_request) if per_request == 1 else k)
    keys = np.concatenate(keys)
    koff = np.arange(requests + 1, dtype=np.int64) * per_request
    coff = np.concatenate([[0], np.cumsum([c.size for c in caches])]).astype(np.int64)
    want = oracle.prefix_match(keys, koff, held, coff)
    got = [torch.full(w.shape, -7, dtype=torch.int32, device="cuda:0") for w in want]
    ws = torch.empty(B.mc_prefix_match_workspace_bytes(requests, len(caches)), dtype=torch.uint8, device="cuda:0")
    B.mc_prefix_match(dev(keys.view(np.int64)), koff.tolist(), dev(held.view(np.int64)), coff.tolist(), *got, ws)
    torch.cuda.synchronize()
    for g, w in zip(got, want):
        np.testing.assert_array_equal(g.cpu().numpy(), w)
