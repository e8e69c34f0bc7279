"""GPU parity of the page order on both sides of the lengths from which fewer threads share a position."""
import numpy as np
import pytest
import torch

from paper_2407_00079_amd import binding as B

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [15, 16, 17, 1023, 1024, 8191, 8192, 8193, 32768, 32769])
@pytest.mark.parametrize("span", [1, 40, 1 << 20, (1 << 31) - 1])
def test_order_matches_oracle(oracle, n, span):
    rng = np.random.default_rng(n + span % 97)
    ids = rng.integers(0, span, size=n, dtype=np.int64).astype(np.int32)
    order = torch.full((n,), -1, dtype=torch.int32, device="cuda:0")
    B.mc_kv_page_order(torch.from_numpy(ids).to("cuda:0"), n, order)
    torch.cuda.synchronize()
    np.testing.assert_array_equal(order.cpu().numpy(), oracle.kv_page_order(ids))
