"""GPU parity of the prefix keys at the lines between the kernels that compute them (one launch for requests of few blocks;
digests and chains in stages for long ones), bit for bit against the CPU oracle."""
import numpy as np
import pytest

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
