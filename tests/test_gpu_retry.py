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
    ew = gen.integers(0, 9, size=m).astype(np.uint32)
    monkeypatch.setenv("CSAW_CHAIN_SPINS", looks)
    g = csaw.Graph(rp, dst, ew)
    monkeypatch.delenv("CSAW_CHAIN_SPINS")
    offs = np.arange(instances + 1, dtype=np.int64) * 2000
    seeds = gen.integers(0, n, size=2000 * instances).astype(np.int32)
    refs = [oracle.sample(rp, dst, ew, offs, seeds, np.array([4, 7, 3], dtype=np.int32), bias_kind=kind, rng_seed=122)
            for kind in (csaw.UNIFORM, csaw.EDGE_WEIGHT)]
    return g, offs, seeds, refs


def same(got, ref):
    np.testing.assert_array_equal(got.offsets.cpu().numpy(), ref.offsets)
    np.testing.assert_array_equal(got.src.cpu().numpy(), ref.src)
    np.testing.assert_array_equal(got.dst.cpu().numpy(), ref.dst)


@pytest.mark.parametrize("looks", ["0", "1"])
def test_sparse_build_gives_up(monkeypatch, csaw, looks):
    """Above 2^20 bitmap words: the compaction's chain gives up (no look), or blocks of either chain may (one)."""
    g, offs, seeds, (ref, _) = case(monkeypatch, csaw, 22, 9, looks)
    for rep in range(3):
        print("[case] retry sparse looks=%s rep=%d" % (looks, rep), flush=True)
        same(g.sample(offs, seeds, [4, 7, 3], rng_seed=122), ref)


@pytest.mark.parametrize("log,instances", [(14, 1), (14, 40), (20, 5), (22, 9)])
def test_second_try(monkeypatch, csaw, log, instances):
    """Builds of 2, 80 and 640 blocks, and a sparse one: pooled calls, unbiased and
    weighted in turn on one workspace, and calls in the library's own scratch."""
    import torch
    g, offs, seeds, refs = case(monkeypatch, csaw, log, instances)
    dev = torch.from_numpy(seeds).cuda()
    cap = g.sample_bound(offs, [4, 7, 3])
    for rep in range(2):
        for kind in (csaw.UNIFORM, csaw.EDGE_WEIGHT):
            print("[case] retry 2^%d x %d kind=%d rep=%d" % (log, instances, kind, rep), flush=True)
            same(g.sample(offs, seeds, [4, 7, 3], kind, rng_seed=122), refs[kind])
            out = (torch.empty(cap, dtype=torch.int32, device="cuda"), torch.empty(cap, dtype=torch.int32, device="cuda"),
                   torch.empty(3 * instances + 1, dtype=torch.int64, device="cuda"))
            same(g.sample_noalloc(offs, dev, [4, 7, 3], out, kind, rng_seed=122), refs[kind])


def test_served_second_try(monkeypatch, csaw):
    """Batches of a server on such a graph: every request is served, with the oracle's edges."""
    g, offs, seeds, (ref, _) = case(monkeypatch, csaw, 20, 5)
    server = csaw.Server(g, num_streams=2, max_batch=4, memory_budget_bytes=1 << 30)
    print("[case] retry served", flush=True)
    tickets = [server.submit_sample(seeds[offs[i]:offs[i + 1]], [4, 7, 3], rng_seed=122, request_id=i) for i in range(5)]
    for i, t in enumerate(tickets):
        r = server.wait(t)
        assert r.status == 0
        at = [slice(ref.offsets[l * 5 + i], ref.offsets[l * 5 + i + 1]) for l in range(3)]
        np.testing.assert_array_equal(r.src, np.concatenate([ref.src[a] for a in at]))
        np.testing.assert_array_equal(r.dst, np.concatenate([ref.dst[a] for a in at]))
    server.close()
