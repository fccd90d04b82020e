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


@pytest.mark.parametrize("Q", [63, 8193, 9000, 33000, 82000, 131072, 131073])
def test_rank_with_nan_is_a_permutation(Q):
    """NaN is outside the contract, but a garbage index must not leave entries of
    the order unwritten (a queue reads them as slots): every method gives the
    stable order of the monotone bits. 0x7fffffff has the bits of the padding."""
    rng = np.random.default_rng(Q)
    u = rng.lognormal(8, 2, Q).astype(np.float32).view(np.uint32)
    bits = np.array([0x7FFFFFFF, 0x7FC00000, 0xFFC00000, 0xFFFFFFFF, 0x7F800000, 0x80000000], dtype=np.uint32)
    some = rng.random(Q) < 0.05
    u[some] = rng.choice(bits, size=int(some.sum()))
    u[[0, Q - 1]] = 0x7FFFFFFF
    for v in (u, np.full(Q, 0x7FFFFFFF, dtype=np.uint32)):
        z = np.where(v == 0x80000000, 0, v).astype(np.uint32)
        key = np.where(z & 0x80000000, ~z, z | 0x80000000).astype(np.uint32)
        ws = torch.full((sage.rank_workspace_bytes(Q),), 0xA5, dtype=torch.uint8, device="cuda")
        order = sage.rank(torch.from_numpy(v.view(np.float32)).cuda(), workspace=ws)
        torch.cuda.synchronize()
        assert np.array_equal(order.cpu().numpy(), np.argsort(key, kind="stable"))
