"""The queue order (Sec. 3.3, smaller index first, ties by request number) at
the sizes where the rank changes its method or fills its tiles: one counting
launch, merged tiles of 512 and 1,024 requests, the radix sort. Exact."""
import numpy as np
import pytest
import torch

from paper_2603_07917_amd import sage
from tests import parity

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("Q", [8192, 8193, 8704, 16385, 32768, 32769, 33793, 66048, 81920, 81921, 131072, 131073])
def test_rank_paths(Q):
    rng = np.random.default_rng(Q)
    cases = [rng.lognormal(8, 3, size=Q),                                  # wide range, few ties
             np.round(rng.uniform(0, 40, size=Q)),                         # ties across every tile
             np.sort(rng.uniform(-5, 5, size=Q))[::-1],                    # descending: tiles in reverse
             np.full(Q, np.inf), np.where(rng.random(Q) < 0.5, -0.0, 0.0)]
    cases[0][rng.random(Q) < 0.2] = np.inf
    cases[2][::7] = -np.inf
    for g in cases:
        g = np.ascontiguousarray(g, dtype=np.float32)
        ws = torch.full((sage.rank_workspace_bytes(Q),), 0xA5, dtype=torch.uint8, device="cuda")
        order = sage.rank(torch.from_numpy(g).cuda(), workspace=ws)
        torch.cuda.synchronize()
        parity.check_rank(order.cpu().numpy(), g)
