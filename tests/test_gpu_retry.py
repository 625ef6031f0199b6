"""Frontier builds whose chain of blocks gives up on the first try: the call
runs again in order, with the oracle's edges. A limit of no looks at all makes
every build of more than one block give up, whatever else runs."""
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


def case(monkeypatch, csaw, log, instances, looks="0"):
    """A graph whose builds by block index take `looks` looks, and a call with the oracle's result."""
    gen = inputs.rng(121)
    n, m = 1 << log, 1 << 16
    src = np.sort(gen.integers(0, n, size=m))
    dst = gen.integers(0, n, size=m).astype(np.int32)
    rp = np.concatenate([[0], np.cumsum(np.bincount(src, minlength=n))]).astype(np.int64)
    monkeypatch.setenv("CSAW_CHAIN_SPINS", looks)
    g = csaw.Graph(rp, dst)
    monkeypatch.delenv("CSAW_CHAIN_SPINS")
    offs = np.arange(instances + 1, dtype=np.int64) * 2000
    seeds = gen.integers(0, n, size=2000 * instances).astype(np.int32)
    ref = oracle.sample(rp, dst, None, offs, seeds, np.array([4, 7, 3], dtype=np.int32), rng_seed=122)
    return g, offs, seeds, ref


def same(got, ref):
    np.testing.assert_array_equal(got.offsets.cpu().numpy(), ref.offsets)
    np.testing.assert_array_equal(got.src.cpu().numpy(), ref.src)
    np.testing.assert_array_equal(got.dst.cpu().numpy(), ref.dst)


@pytest.mark.parametrize("looks", ["0", "1"])
def test_sparse_build_gives_up(monkeypatch, csaw, looks):
    """Above 2^20 bitmap words: the compaction's chain gives up (no look), or blocks of either chain may (one)."""
    g, offs, seeds, ref = case(monkeypatch, csaw, 22, 9, looks)
    for rep in range(3):
        print("[case] retry sparse looks=%s rep=%d" % (looks, rep), flush=True)
        same(g.sample(offs, seeds, [4, 7, 3], rng_seed=122), ref)
