"""A call that fits the library's own scratch only without a dirty list: 1.2M
bitmap words in dense builds of sixteen words a thread, the last block partly
filled, fixed fanouts and forest fire, first and second try. Against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2009_09103_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("looks", ["", "0"])
def test_scratch_without_dirty_list(monkeypatch, looks):
    import torch
    from paper_2009_09103_amd import csaw
    gen = inputs.rng(151)
    n, m, ni, per = (1 << 22) - 64, 500000, 9, 5035
    src = gen.integers(0, n, size=m)
    src[:m // 4] = gen.integers(0, 300, size=m // 4)
    src.sort()
    dst = gen.integers(0, n, size=m).astype(np.int32)
    dst[::3] = gen.integers(0, 300, size=len(dst[::3]))
    rp = np.concatenate([[0], np.cumsum(np.bincount(src, minlength=n))]).astype(np.int64)
    ew = gen.integers(0, 9, size=m).astype(np.uint32)
    assert np.diff(rp).max() >= 64
    monkeypatch.setenv("CSAW_CHAIN_SPINS", looks)
    g = csaw.Graph(rp, dst, ew)
    offs = np.arange(ni + 1, dtype=np.int64) * per
    seeds = gen.integers(0, n, size=ni * per).astype(np.int32)
    seeds[::10] = gen.integers(0, 300, size=len(seeds[::10]))
    dev = torch.from_numpy(seeds).cuda()
    cap = g.sample_bound(offs, [64, 1])
    out = (torch.empty(cap, dtype=torch.int32, device="cuda"), torch.empty(cap, dtype=torch.int32, device="cuda"),
           torch.empty(2 * ni + 1, dtype=torch.int64, device="cuda"))
    for kind, burn in ((csaw.UNIFORM, 0), (csaw.EDGE_WEIGHT, 0), (csaw.UNIFORM, int(0.7 * 2 ** 32))):
        print("[case] scratch looks=%s kind=%d burn=%d" % (looks or "default", kind, burn), flush=True)
        ref = oracle.sample(rp, dst, ew, offs, seeds, np.array([64, 1], dtype=np.int32), bias_kind=kind, rng_seed=152, burn=burn)
        got = g.sample_noalloc(offs, dev, [64, 1], out, kind, rng_seed=152, burn=burn)
        assert got.num_edges == ref.num_edges
        np.testing.assert_array_equal(got.offsets.cpu().numpy(), ref.offsets)
        np.testing.assert_array_equal(got.src.cpu().numpy(), ref.src)
        np.testing.assert_array_equal(got.dst.cpu().numpy(), ref.dst)
