"""Layer sampling where its routes change: seed sets around the 64 lanes, the runs a
lane sums and the largest set; lists around the four weights of a load, the
512 of the scan and the chunk tables; fanouts about the number of positive
lists; the same picks with and without the walk guide. Against the oracle."""
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


def stair_graph():
    """Lists of 1 to 40 edges, of 508 to 516 and of up to 3,000, each vertex's in random order of weights."""
    gen = inputs.rng(95)
    n = 4096
    deg = gen.integers(1, 41, size=n)
    deg[gen.random(n) < 0.3] = 0
    deg[::37] = np.resize([508, 511, 512, 513, 516, 1023, 1024, 1025, 3000], len(deg[::37]))
    rp = np.concatenate([[0], np.cumsum(deg)]).astype(np.int64)
    col = np.concatenate([np.sort(gen.choice(n, size=d, replace=False)) for d in deg]).astype(np.int32)
    return rp, col, gen


@pytest.mark.parametrize("guide", [False, True])
@pytest.mark.parametrize("kind", ["edge_weight", "wide", "neighbor_degree"])
def test_layer_routes(csaw, kind, guide):
    rp, col, gen = stair_graph()
    n = len(rp) - 1
    ew = gen.integers(0, 9, size=len(col)) * (gen.random(len(col)) < 0.6)
    if kind == "wide":
        ew = gen.integers((1 << 32) - 9, 1 << 32, size=len(col), dtype=np.uint64)
    ew = ew.astype(np.uint32)
    bias = csaw.NEIGHBOR_DEGREE if kind == "neighbor_degree" else csaw.EDGE_WEIGHT
    g = csaw.Graph(rp, col, ew)
    if guide:  # a walk builds it
        g.walk(np.zeros(1, dtype=np.int32), 1, bias)
    sizes = [1, 2, 3, 5, 9, 63, 64, 65, 511, 512, 513, 1025, 2048]
    sets = [np.sort(gen.choice(n, size=k, replace=False)) for k in sizes]
    offs = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    seeds = np.concatenate(sets).astype(np.int32)
    for fan, rounds in (([64, 64, 64], 0), ([5, 3, 2, 1], 0), ([64], -1), ([33, 64], 1)):
        print("[case] layer %s guide=%s fan=%s rounds=%d" % (kind, guide, fan, rounds), flush=True)
        src, dst, counts = g.layer_sample(offs, seeds, fan, bias, rng_seed=96, instance_base=4, rounds=rounds)
        rs, rd, rc = oracle.layer_sample(rp, col, ew, offs, seeds, fan, bias_kind=bias, rng_seed=96, instance_base=4,
                                         rounds={-1: 0, 0: 8}.get(rounds, rounds))
        np.testing.assert_array_equal(counts.cpu().numpy(), rc)
        np.testing.assert_array_equal(src.cpu().numpy(), rs)
        np.testing.assert_array_equal(dst.cpu().numpy(), rd)
