"""Tables that calls built to draw faster (walk guides, hop table, rank index)
go where a call cannot get its memory otherwise: a workspace whose allocator has
none at first. The call and those after it give the oracle's results, and so do
weighted walks on a graph that gave its guide back."""
import numpy as np
import pytest

import oracle
from paper_2009_09103_amd import inputs

pytestmark = pytest.mark.gpu


def test_tables_go_for_a_workspace():
    import torch
    from paper_2009_09103_amd import csaw
    rp, col = inputs.rmat_csr(16, 32 << 16, 131, symmetrize=True)
    ew = inputs.dst_outdeg_weights(rp, col)
    g = csaw.Graph(rp, col, ew)
    starts = inputs.walker_starts(rp, col, 3000, 132)
    offs, seeds = inputs.single_instance_seeds(rp, col, 500, 133)
    want = {b: oracle.walk(rp, col, ew, starts[:300], 40, bias_kind=b, rng_seed=134, node2vec=(1, 2, 4))[0] for b in (0, 1, 3)}
    ref = oracle.sample(rp, col, ew, offs, seeds, np.array([20, 10], dtype=np.int32), bias_kind=1, rng_seed=135)

    def walks():
        for b in (0, 1, 3):
            nw = 3000 if b < 3 else 300
            paths, _ = g.walk(starts[:nw], 40, b, rng_seed=134, node2vec=(1, 2, 4))
            np.testing.assert_array_equal(paths.cpu().numpy()[:300], want[b])

    refused, kept = [], {}

    def alloc(nbytes):
        if not refused:
            refused.append(nbytes)
            return 0
        t = torch.empty(nbytes, dtype=torch.uint8, device="cuda")
        kept[t.data_ptr()] = t
        return t.data_ptr()

    for _ in range(20):  # enough steps for the hop table
        walks()
    print("[case] give back: a workspace of a graph with every table", flush=True)
    csaw.set_allocator(alloc, lambda p: kept.pop(p, None))
    try:
        torch.cuda.synchronize()
        before = torch.cuda.mem_get_info()[0]
        res = g.sample(offs, seeds, [20, 10], csaw.EDGE_WEIGHT, rng_seed=135)
        torch.cuda.synchronize()
        assert refused and torch.cuda.mem_get_info()[0] > before + 80 * len(col) // 2
        np.testing.assert_array_equal(res.src.cpu().numpy(), ref.src)
        np.testing.assert_array_equal(res.dst.cpu().numpy(), ref.dst)
        np.testing.assert_array_equal(res.offsets.cpu().numpy(), ref.offsets)
        walks()
        res = g.sample(offs, seeds, [20, 10], csaw.EDGE_WEIGHT, rng_seed=135)
        np.testing.assert_array_equal(res.dst.cpu().numpy(), ref.dst)
        g.close()
    finally:
        csaw.set_allocator(None, None)
