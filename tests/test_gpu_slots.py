"""The slot-per-lane selection kernel at the sizes where its packing, staging
and search routes change, against the oracle, element by element: fanouts that
fill a wavefront's 64 lanes exactly, straddle it or leave one lane over; lists
at the staging bounds (8 candidates per slot, the LDS words of a wavefront),
at the longest list a lane scans and past 512; zero weights, weights whose
total needs 64 bits, lists hardly longer than the fanout (direct draws); every
count of rounds; before the walk guide exists, with it and with it off."""
import numpy as np
import pytest

import oracle
from paper_2009_09103_amd import inputs

pytestmark = pytest.mark.gpu

LENGTHS = [1, 2, 5, 6, 8, 9, 10, 31, 32, 33, 39, 40, 41, 63, 64, 65, 79, 80, 81, 127, 128, 129, 219, 220, 221, 367, 368,
           369, 511, 512, 513, 700, 1025]


@pytest.fixture(scope="module")
def csaw():
    import torch
    assert torch.cuda.is_available()
    from paper_2009_09103_amd import csaw as c
    return c


def graph(weights):
    gen = inputs.rng(77)
    n = 1500
    deg = np.array([LENGTHS[i % len(LENGTHS)] for i in range(n)], dtype=np.int64)
    rp = np.concatenate([[0], np.cumsum(deg)]).astype(np.int64)
    col = np.concatenate([np.sort(gen.choice(n, size=d, replace=False)) for d in deg]).astype(np.int32)
    m = len(col)
    if weights == "plain":
        ew = gen.integers(1, 100, size=m)
    elif weights == "zeros":  # about half zero, some lists all zero
        ew = gen.integers(0, 50, size=m) * (gen.random(m) < 0.5)
        ew[rp[9]:rp[10]] = 0
    elif weights == "skewed":  # a few candidates hold nearly all of the weight
        ew = np.where(gen.random(m) < 0.05, 1 << 24, 1)
    else:  # totals of 64 bits
        ew = gen.integers((1 << 32) - 1000, 1 << 32, size=m, dtype=np.uint64)
    return rp, col, ew.astype(np.uint32)


@pytest.mark.parametrize("rounds", [0, 1, -1])
@pytest.mark.parametrize("weights", ["plain", "zeros", "skewed", "wide"])
def test_slot_routes(csaw, weights, rounds):
    rp, col, ew = graph(weights)
    n = len(rp) - 1
    fans = [[1, 2], [5, 3], [10, 1], [21, 0], [22, 0], [32, 2], [63, 0], [64, 1], [-1, 1]]
    offs = np.arange(len(fans) * 3 + 1, dtype=np.int64) * 97
    gen = inputs.rng(78)
    seeds = np.concatenate([gen.choice(n, size=97, replace=False) for _ in range(len(offs) - 1)]).astype(np.int32)
    fan = np.array([fans[i % len(fans)] for i in range(len(offs) - 1)], dtype=np.int32)
    bias = np.array([(0, 1, 2)[i // len(fans)] for i in range(len(offs) - 1)], dtype=np.int32)
    orc_rounds = {-1: 0, 0: 8}.get(rounds, rounds)
    ref = oracle.sample(rp, col, ew, offs, seeds, fan, bias_kinds=bias, rng_seed=5, rounds=orc_rounds)
    g = csaw.Graph(rp, col, ew)

    def check(what):
        print("[case] slots %s rounds=%d %s" % (weights, rounds, what), flush=True)
        res = g.sample(offs, seeds, fan, bias, rng_seed=5, rounds=rounds)
        np.testing.assert_array_equal(res.offsets.cpu().numpy(), ref.offsets)
        np.testing.assert_array_equal(res.src.cpu().numpy(), ref.src)
        np.testing.assert_array_equal(res.dst.cpu().numpy(), ref.dst)

    check("no guide")
    g.walk(seeds[:1], 1, csaw.EDGE_WEIGHT)  # builds the guide of one weight array
    check("edge-weight guide only")
    g.walk(seeds[:1], 1, csaw.NEIGHBOR_DEGREE)
    check("both guides")
    g.set_walk_guides(False)
    g.set_tuning(0, 0)
    check("guides and scanned lists off")


def test_guide_appears_after_enough_draws(csaw):
    """Weighted sampling builds the guide itself once its draws have paid for
    it: the same edges before, at and after that call."""
    rp, col = inputs.rmat_csr(13, 8 << 13, 81)
    offs, seeds = inputs.single_instance_seeds(rp, col, 600, 82)
    ref = oracle.sample(rp, col, None, offs, seeds, [25, 10], bias_kind=2, rng_seed=9)
    g = csaw.Graph(rp, col)
    assert ref.num_edges * 20 > len(col)
    for _ in range(20):
        res = g.sample(offs, seeds, [25, 10], csaw.NEIGHBOR_DEGREE, rng_seed=9)
        np.testing.assert_array_equal(res.dst.cpu().numpy(), ref.dst)
        np.testing.assert_array_equal(res.src.cpu().numpy(), ref.src)
