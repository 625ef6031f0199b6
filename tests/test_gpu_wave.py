"""Weighted calls before their guide is built with both bounds at zero: one
wavefront per list, take-all lists among them (shorter than the fanout, and whole
neighborhoods), zero weights, lists around 64 to 512. Against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2009_09103_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fanouts", [[64, 5], [3, 40, 2], [-1, 4]])
@pytest.mark.parametrize("kind", ["edge_weight", "zeros", "neighbor_degree"])
def test_wave_route(kind, fanouts):
    from paper_2009_09103_amd import csaw
    rp, col = inputs.rmat_csr(13, 24 << 13, 102)
    assert np.diff(rp).max() > 512
    gen = inputs.rng(103)
    ew = gen.integers(0, 40, size=len(col)) * (gen.random(len(col)) < (0.5 if kind == "zeros" else 1.0))
    ew = ew.astype(np.uint32)
    g = csaw.Graph(rp, col, ew)
    g.set_tuning(0, 0)
    bias = csaw.NEIGHBOR_DEGREE if kind == "neighbor_degree" else csaw.EDGE_WEIGHT
    offs = np.array([0, 40, 41, 200], dtype=np.int64)
    seeds = gen.integers(0, len(rp) - 1, size=200).astype(np.int32)
    print("[case] wave %s fanouts=%s" % (kind, fanouts), flush=True)
    ref = oracle.sample(rp, col, ew, offs, seeds, fanouts, bias_kind=bias, rng_seed=104)
    for _ in range(2):
        res = g.sample(offs, seeds, fanouts, bias, rng_seed=104)
        np.testing.assert_array_equal(res.offsets.cpu().numpy(), ref.offsets)
        np.testing.assert_array_equal(res.src.cpu().numpy(), ref.src)
        np.testing.assert_array_equal(res.dst.cpu().numpy(), ref.dst)
