"""Unbiased steps through the hop table, which a graph builds once its calls have
asked for enough of them: walks before and after it exists, at path lengths
around the run a lane keeps before it stores, with restarts, jumps, sinks and
Metropolis-Hastings proposals; multi-dimensional walks at the bounds of their
LDS layout (degrees that 16 bits do not hold, totals that need 64 bits).
Every entry against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2009_09103_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def csaw():
    import torch
    assert torch.cuda.is_available()
    from paper_2009_09103_amd import csaw as c
    return c


@pytest.mark.parametrize("length", [1, 31, 63, 64, 65, 128, 130])
@pytest.mark.parametrize("bias,restart,jump", [(0, 0, 0), (0, 1 << 29, 1 << 28), (4, 0, 0), (4, 1 << 28, 1 << 28)])
def test_walks_before_and_after_the_table(csaw, length, bias, restart, jump):
    rp, col = inputs.rmat_csr(12, 4 << 12, 91)  # directed: walks end at sinks
    g = csaw.Graph(rp, col)
    for nw in (3, 5000):  # the first call is too small for the table, the second pays for it
        assert (nw * length < len(col) // 2) == (nw == 3) or length == 1
        starts = inputs.walker_starts(rp, col, nw, 92)
        print("[case] hops length=%d bias=%d walkers=%d" % (length, bias, nw), flush=True)
        paths, steps = g.walk(starts, length, bias, rng_seed=93, walker_base=5, restart=restart, jump=jump)
        ref, rs, _ = oracle.walk(rp, col, None, starts, length, bias_kind=bias, rng_seed=93, walker_base=5,
                                 restart=restart, jump=jump)
        np.testing.assert_array_equal(paths.cpu().numpy(), ref)
        assert steps == int(rs.sum())


def star(d):
    """Vertex 0 and d leaves, edges both ways, and one edge between two leaves."""
    deg = np.concatenate([[d], np.ones(d, dtype=np.int64)])
    deg[1] = 2
    rp = np.concatenate([[0], np.cumsum(deg)]).astype(np.int64)
    col = np.zeros(rp[-1], dtype=np.int32)
    col[:d] = np.arange(1, d + 1)
    col[d + 1] = 2
    return rp, col


@pytest.mark.parametrize("d,hub_slots", [(65534, 3), (65535, 3), (70000, 40), (2_200_000, 2000)])
def test_pools_with_hubs(csaw, d, hub_slots):
    """Hub degrees around 2^16, and a pool whose degree total passes 2^32."""
    rp, col = star(d)
    g = csaw.Graph(rp, col)
    gen = inputs.rng(94)
    sizes = [2048, 2000, 65, 1]
    pools = []
    for k in sizes:
        p = gen.integers(1, d + 1, size=k)
        p[:min(k, hub_slots)] = 0
        pools.append(gen.permutation(p))
    po = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    pool = np.concatenate(pools).astype(np.int32)
    if hub_slots == 2000:
        assert hub_slots * d > 1 << 32
    for budget in (20, 130):
        print("[case] hops mdrw hub=%d budget=%d" % (d, budget), flush=True)
        src, dst, steps, total = g.mdrw(po, pool, budget, rng_seed=95, instance_base=3)
        rs, rd, rst = oracle.mdrw(rp, col, po, pool, budget, rng_seed=95, instance_base=3)
        np.testing.assert_array_equal(src.cpu().numpy(), rs)
        np.testing.assert_array_equal(dst.cpu().numpy(), rd)
        np.testing.assert_array_equal(steps.cpu().numpy(), rst)
        assert total == int(rst.sum())
    # enough steps for the table on the largest graph too
    many = np.tile(np.array([0, 1], dtype=np.int32), 400)
    off = np.arange(401, dtype=np.int64) * 2
    src, dst, steps, _ = g.mdrw(off, many, 600, rng_seed=96)
    rs, rd, rst = oracle.mdrw(rp, col, off, many, 600, rng_seed=96)
    np.testing.assert_array_equal(src.cpu().numpy(), rs)
    np.testing.assert_array_equal(dst.cpu().numpy(), rd)
