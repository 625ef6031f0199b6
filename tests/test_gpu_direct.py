"""Direct draws alone from weighted lists without a guide: no list is scanned by
a lane whatever the bounds are, beside unbiased instances and take-all lists.
Against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2009_09103_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bounds", [(16, 32), (0, 32), (0, 0)])
@pytest.mark.parametrize("mixed", [False, True])
def test_direct_only(mixed, bounds):
    from paper_2009_09103_amd import csaw
    rp, col = inputs.rmat_csr(12, 20 << 12, 181)
    deg = np.diff(rp)
    assert deg.max() > 512 and all((deg == d).any() for d in (1, 8, 16, 32, 33))
    gen = inputs.rng(182)
    ew = (gen.integers(0, 40, size=len(col)) * (gen.random(len(col)) < .8)).astype(np.uint32)
    g = csaw.Graph(rp, col, ew)
    g.set_tuning(*bounds)
    offs = np.arange(7, dtype=np.int64) * 120
    seeds = gen.integers(0, len(rp) - 1, size=720).astype(np.int32)
    fan = np.array([[25, 10], [5, 3], [64, 2], [-1, 4], [1, 1], [31, 32]], dtype=np.int32)
    bias = np.array([1, 2, 1, 1, 2, 1], dtype=np.int32)
    if mixed:
        bias[::2] = csaw.UNIFORM
    ref = oracle.sample(rp, col, ew, offs, seeds, fan, bias_kinds=bias, rng_seed=183, rounds=0)
    scopes = {}
    for rep in range(2):
        print("[case] direct mixed=%s bounds=%s rep=%d" % (mixed, bounds, rep), flush=True)
        csaw.profile_reset()
        csaw.profile_enable(rep == 0)
        got = g.sample(offs, seeds, fan, bias, rng_seed=183, rounds=csaw.DIRECT_ONLY)
        csaw.profile_enable(False)
        if rep == 0:
            scopes = {k: csaw.profile_read(k)[1] for k in ("select_slots", "select_wave", "select_big")}
        np.testing.assert_array_equal(got.offsets.cpu().numpy(), ref.offsets)
        np.testing.assert_array_equal(got.src.cpu().numpy(), ref.src)
        np.testing.assert_array_equal(got.dst.cpu().numpy(), ref.dst)
    csaw.profile_reset()
    assert scopes == ({"select_slots": 2, "select_wave": 0, "select_big": 2} if mixed else
                      {"select_slots": 0, "select_wave": 2, "select_big": 2})
