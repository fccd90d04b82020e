"""The index scan (Sec. 3.3) at the edges of its lane layouts: 16, 32 or 64
lanes per row, 1 to 64 bins per lane, rows that fill them or not, batches
that leave the last wave's rows short. Against the oracle; the bound is the
parity bar of the index on identical inputs."""
import numpy as np
import pytest
import torch

import oracle
from paper_2603_07917_amd import sage, workloads
from tests import parity

pytestmark = pytest.mark.gpu


def dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def host(t):
    torch.cuda.synchronize()
    return t.cpu().numpy()


def close(g, G):
    assert np.array_equal(np.isinf(g), np.isinf(G))
    f = np.isfinite(G)
    assert np.all(np.abs(g[f].astype(np.float64) - G[f]) <= parity.INDEX_RTOL * np.abs(G[f]))


@pytest.mark.parametrize("B", [1, 16, 17, 32, 33, 64, 65, 128, 129, 256, 257, 260, 512, 513, 1024, 1025, 1500, 2047, 2048, 2049, 4096])
def test_index_layouts(B):
    rng = np.random.default_rng(B)
    Q = 133
    mass = rng.dirichlet(np.full(B, 0.3), size=Q).astype(np.float32)
    mass[rng.random((Q, B)) < 0.5] = 0.0
    mass[5] = 0.0                                             # no mass: +inf
    plen = rng.integers(0, 4000, size=Q).astype(np.int32)
    _, r = workloads.log_bins(16384, B)
    x = oracle.cost(plen, r)
    G, arg = oracle.gittins(mass.astype(np.float64), x)
    md, pd, rd = dev(mass), dev(plen), dev(r)
    g, a = sage.index(md, pd, rd, with_argmin=True)
    g, a = host(g), host(a)
    close(g, G)
    ratio = g.astype(np.float64)
    assert a[5] == -1 and np.all((a >= 0) == np.isfinite(ratio))
    for q in (1, 2, 3, 5):                                    # fewer rows than a wave holds
        assert np.array_equal(host(sage.index(md[:q].contiguous(), pd[:q].contiguous(), rd)).view(np.uint32),
                              g[:q].view(np.uint32))
    gen = rng.integers(0, 2000, size=Q).astype(np.int32)
    Ga, _ = oracle.gittins_attained(mass.astype(np.float64), x, oracle.attained_service(plen, gen, 200))
    close(host(sage.index_attained(md, pd, rd, dev(gen), 200)), Ga)
    levels = 70                                               # past one block of 64 levels
    table = host(sage.index_attained_table(md, pd, rd, levels, 250))
    for lv in (0, 1, 3, 63, 64, 69):
        Gt, _ = oracle.gittins_attained(mass.astype(np.float64), x,
                                        oracle.attained_service(plen, np.full(Q, lv * 250), 250))
        close(table[lv], Gt)
        one = host(sage.index_attained(md, pd, rd, dev(np.full(Q, lv * 250, np.int32)), 250))
        assert np.array_equal(table[lv].view(np.uint32), one.view(np.uint32)), lv
    mean = host(sage.index_variant(md, pd, rd, kind="mean", noise=0.2))
    assert np.array_equal(np.isinf(mean), mass.sum(axis=1) == 0)


@pytest.mark.parametrize("B", [1, 40, 64, 200, 256, 301, 512, 513, 1024, 2048])
@pytest.mark.parametrize("Q,levels", [(1, 1), (1, 70), (3, 131), (9, 5), (70, 6), (133, 2), (1030, 3)])
def test_table_shares_and_few_levels(B, Q, levels):
    """The refresh table where a few rows' levels are shared between workgroups
    (with a share that starts inside a block of 64 levels) and where it has so
    few levels that rows take the lanes: the bits of the per-level calls, past a
    row's last outcome too."""
    rng = np.random.default_rng(B + Q + levels)
    mass = rng.dirichlet(np.full(B, 0.3), size=Q).astype(np.float32)
    mass[rng.random((Q, B)) < 0.5] = 0.0
    mass[Q // 2, :] = 0.0                                     # no mass at all
    if Q > 2:
        mass[2, B // 3:] = 0.0                                # done after a few levels
    plen = rng.integers(0, 4000, size=Q).astype(np.int32)
    _, r = workloads.log_bins(16384, B)
    md, pd, rd = dev(mass), dev(plen), dev(r)
    bucket = max(1, 20000 // levels)
    table = host(sage.index_attained_table(md, pd, rd, levels, bucket, out=torch.full((levels, Q), 7.0, device="cuda")))
    for lv in range(levels):
        one = host(sage.index_attained(md, pd, rd, dev(np.full(Q, lv * bucket, np.int32)), bucket))
        assert np.array_equal(table[lv].view(np.uint32), one.view(np.uint32)), lv
    Gt, _ = oracle.gittins_attained(mass.astype(np.float64), oracle.cost(plen, r),
                                    oracle.attained_service(plen, np.full(Q, (levels // 2) * bucket), bucket))
    close(table[levels // 2], Gt)


@pytest.mark.parametrize("B", [3, 31, 67, 102, 127, 200, 255, 301, 511, 515, 700, 1023, 1100])
def test_given_cost_rows_of_any_width(B):
    """Rows whose bins do not fill their lanes, masses and costs loaded four at a
    time from any 4-byte aligned place; the last row ends its buffer."""
    rng = np.random.default_rng(B)
    Q = 37
    mass = rng.dirichlet(np.full(B, 0.3), size=Q).astype(np.float32)
    cost = np.sort(rng.lognormal(8, 2, size=(Q, B)), axis=1).astype(np.float32)
    G, arg = oracle.gittins(mass.astype(np.float64), cost)
    g, a = sage.index(dev(mass), cost=dev(cost), with_argmin=True)
    close(host(g), G)
    assert np.all(host(a) >= 0)
    assert np.array_equal(host(sage.index(dev(mass), cost=dev(cost))).view(np.uint32), host(g).view(np.uint32))


@pytest.mark.parametrize("B", [16, 300])
def test_table_of_the_most_levels(B):
    """levels * bucket = 2^31 - 1: four (B = 16) or two levels at a time would
    count past the 32-bit range in the last step. Done after 16,384 levels."""
    levels = 2**31 - 1
    _, r = workloads.log_bins(16384, B)
    md, pd, rd = dev(np.full((1, B), 1.0 / B, np.float32)), dev(np.array([100], np.int32)), dev(r)
    table = sage.index_attained_table(md, pd, rd, levels, 1).view(-1)
    for lv in (0, 1, 63, 64, 8191, 16000):
        one = host(sage.index_attained(md, pd, rd, dev(np.array([lv], np.int32)), 1))
        assert np.array_equal(host(table[lv:lv + 1]).view(np.uint32), one.view(np.uint32)), lv
    done = int(np.ceil(r[-1]))
    assert bool(torch.isinf(table[done:]).all()) and bool(torch.isfinite(table[:int(r[-1])]).all())
