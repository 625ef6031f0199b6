"""node2vec on graphs whose edges to the previous vertex are repeated: runs of its
copies inside a chunk of 64 entries, across one boundary and across several, in
the shorter list and in the longer one, self loops among them, each bias the
largest and zero in turn. Every path against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2009_09103_amd import inputs

pytestmark = pytest.mark.gpu


def graph(copies):
    gen = inputs.rng(191)
    n = 400
    pairs = [(0, 1)] * copies + [(0, 2)] * 63 + [(1, 2)] * 64 + [(0, 0)] * (copies // 2) + [(2, 3)] * (copies + 65) + [(3, 4)] * 130
    for v in range(5):
        pairs += [(v, int(x)) for x in gen.integers(5, n, size=90 * (v + 1))]
    pairs += [(int(a), int(b)) for a, b in gen.integers(5, n, size=(1500, 2))]
    a = np.array(pairs)
    a = np.concatenate([a, a[:, ::-1]])
    a = a[np.lexsort((a[:, 1], a[:, 0]))]
    rp = np.concatenate([[0], np.cumsum(np.bincount(a[:, 0], minlength=n))]).astype(np.int64)
    return rp, a[:, 1].astype(np.int32)


@pytest.mark.parametrize("weights", [(4, 2, 1), (1, 2, 4), (9, 1, 1), (0, 1, 1), (1, 0, 1), (1, 1, 0), (1, 0, 0), (3, 4, 5)])
@pytest.mark.parametrize("copies", [1, 2, 40, 64, 200, 700])
def test_copies_of_the_previous_vertex(copies, weights):
    from paper_2009_09103_amd import csaw
    rp, col = graph(copies)
    g = csaw.Graph(rp, col)
    starts = np.concatenate([np.arange(5).repeat(40), inputs.rng(192).integers(0, len(rp) - 1, size=100)]).astype(np.int32)
    print("[case] rank repeats copies=%d weights=%s" % (copies, weights), flush=True)
    paths, steps = g.walk(starts, 24, csaw.NODE2VEC, rng_seed=193, node2vec=weights)
    ref, rs, _ = oracle.walk(rp, col, None, starts, 24, bias_kind=oracle.NODE2VEC, rng_seed=193, node2vec=weights)
    np.testing.assert_array_equal(paths.cpu().numpy(), ref)
    assert steps == int(rs.sum())
