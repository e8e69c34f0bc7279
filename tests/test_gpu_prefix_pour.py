"""GPU parity of the prefix keys of a queue of long prompts, bit for bit against the oracle: requests that end before, at and
after the block from which their own compute unit digests (csrc/prefix_hash.hip: prefix_pour_kernel), groups of 16 digests
that end early, and the lines to the launches by ranges."""
import numpy as np
import pytest

from test_gpu_prefix import gpu_keys

pytestmark = pytest.mark.gpu


# tokens of a block, blocks per request
@pytest.mark.parametrize("bt,blocks", [
    (512, [63, 64, 65, 79, 80, 81, 130, 0, 1, 16] + [105] * 57),         # the compute unit's own from block 64 on
    (512, [300, 1] + [100] * 60),
    (16, [1, 15, 16, 17, 33, 0, 127] + [111] * 60),                      # all blocks its own
    (16, [4096] + [50] * 50), (16, [4097] + [50] * 50),                  # as many as the LDS has room for, and one more
    (16, [33] * 200), (16, [33] * 256), (16, [34] * 257),                # as many requests as compute units, and one more
])
def test_keys_of_a_queue_match_oracle(oracle, bt, blocks):
    print(f"prefix pour case bt={bt} blocks={blocks[:7]} of {len(blocks)}", flush=True)
    assert sum(blocks) >= 6250                     # a queue: digests for several microseconds of the whole chip
    rng = np.random.default_rng(sum(blocks) + bt)
    lens = [max(n * bt - (r % 3) * (bt // 3), 0) for r, n in enumerate(blocks)]
    tokens = rng.integers(-5, 128000, size=sum(lens), dtype=np.int32)
    off = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
    ref, _ = oracle.prefix_hash(tokens, off, bt)
    for _ in range(2):
        np.testing.assert_array_equal(gpu_keys(tokens, off, bt), ref)
