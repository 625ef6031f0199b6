"""Calls of one shape and one set of buffers that change their instances' bias
kinds, both bounds at zero and no guide yet: all weighted, then some unbiased,
then all weighted again, each against the oracle. A launch sequence captured for
the first kind of call holds a kernel that draws by weight alone."""
import numpy as np
import pytest

import oracle
from paper_2009_09103_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["edge_weight", "neighbor_degree"])
def test_bias_kinds_change_between_calls(kind):
    import torch
    from paper_2009_09103_amd import csaw
    rp, col = inputs.rmat_csr(12, 16 << 12, 111)
    assert np.diff(rp).max() > 512
    gen = inputs.rng(112)
    ew = gen.integers(0, 40, size=len(col)).astype(np.uint32)
    g = csaw.Graph(rp, col, ew)
    g.set_tuning(0, 0)
    bias = csaw.NEIGHBOR_DEGREE if kind == "neighbor_degree" else csaw.EDGE_WEIGHT
    offs = np.arange(9, dtype=np.int64) * 6
    seeds = gen.integers(0, len(rp) - 1, size=48).astype(np.int32)
    seeds[::6] = int(np.argmax(np.diff(rp)))
    fanouts = np.array([[5, 3]] * 8, dtype=np.int32)
    weighted = np.full(8, bias, dtype=np.int32)
    mixed = np.where(np.arange(8) % 2 == 0, csaw.UNIFORM, bias).astype(np.int32)
    cap = g.sample_bound(offs, fanouts, weighted)
    dev_seeds = torch.from_numpy(seeds).cuda()
    out = (torch.empty(cap, dtype=torch.int32, device="cuda"), torch.empty(cap, dtype=torch.int32, device="cuda"),
           torch.empty(17, dtype=torch.int64, device="cuda"))
    for rep in range(2):
        for what, kinds in (("weighted", weighted), ("mixed", mixed), ("weighted", weighted)):
            print("[case] replay %s %s rep=%d" % (kind, what, rep), flush=True)
            res = g.sample(offs, dev_seeds, fanouts, kinds, rng_seed=113, out=out)
            ref = oracle.sample(rp, col, ew, offs, seeds, fanouts, bias_kinds=kinds, rng_seed=113)
            assert res.num_edges == ref.num_edges
            np.testing.assert_array_equal(res.offsets.cpu().numpy(), ref.offsets)
            np.testing.assert_array_equal(res.src.cpu().numpy()[:ref.num_edges], ref.src)
            np.testing.assert_array_equal(res.dst.cpu().numpy()[:ref.num_edges], ref.dst)
