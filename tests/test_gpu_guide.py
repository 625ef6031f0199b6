"""Walk guide buckets where their contents change: edges that fill many
buckets, two positions to a bucket and more, zero weights between them, lists of
one edge, weights near 2^32; walked by one wavefront per walker and by one lane
per walker, at path lengths around the runs that either stores. Every path
against the oracle."""
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


def weights(kind, m, gen):
    if kind == "heavy":  # one edge in 20 fills hundreds of buckets, the others share theirs
        return np.where(gen.random(m) < 0.05, 1 << 22, gen.integers(0, 3, size=m))
    if kind == "zeros":
        return gen.integers(0, 9, size=m) * (gen.random(m) < 0.4)
    if kind == "even":  # every bucket starts where an interval does
        return np.full(m, 64)
    if kind == "steps":  # geometric: most of a list lies in its first bucket
        return 1 << gen.integers(0, 31, size=m)
    return gen.integers((1 << 32) - 9, 1 << 32, size=m, dtype=np.uint64)


@pytest.mark.parametrize("length", [1, 31, 32, 33, 63, 64, 65, 129])
@pytest.mark.parametrize("kind", ["heavy", "zeros", "even", "steps", "wide"])
def test_guide_walks(csaw, kind, length):
    rp, col = inputs.rmat_csr(11, 12 << 11, 83, symmetrize=True)
    deg = np.diff(rp)
    assert (deg == 1).any() and deg.max() > 512
    ew = weights(kind, len(col), inputs.rng(84)).astype(np.uint32)
    g = csaw.Graph(rp, col, ew)
    for nw, moves in ((70, (0, 0)), (70, (1 << 29, 1 << 28)), (12300, (0, 0)), (12300, (1 << 29, 1 << 28))):
        starts = inputs.walker_starts(rp, col, nw, 85)
        print("[case] guide %s length=%d walkers=%d moves=%s" % (kind, length, nw, moves), flush=True)
        paths, steps = g.walk(starts, length, csaw.EDGE_WEIGHT, rng_seed=86, walker_base=3, restart=moves[0], jump=moves[1])
        ids = np.arange(0, nw, 1 if nw < 1000 else 16)
        ref, _, _ = oracle.walk(rp, col, ew, starts[ids], length, bias_kind=oracle.EDGE_WEIGHT, rng_seed=86,
                                walker_ids=ids.astype(np.uint64) + 3, restart=moves[0], jump=moves[1])
        got = paths.cpu().numpy()
        np.testing.assert_array_equal(got[ids], ref)
        assert steps == int((got[:, 1:] >= 0).sum())
