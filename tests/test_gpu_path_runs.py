"""Path entries stored at once (launches of few walkers) and in runs of 64 or 32
(many): unbiased, Metropolis-Hastings and weighted walks on both sides of the
lines between the two, at path lengths around the runs, with restarts and jumps
and walks that end early. Every 97th path against the oracle."""
import numpy as np
import pytest

import oracle
from paper_2009_09103_amd import inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("moves", [(0, 0), (1 << 29, 1 << 28)])
@pytest.mark.parametrize("bias,line", [(0, 98304), (4, 98304), (1, 57344)])
@pytest.mark.parametrize("length", [1, 31, 32, 33, 63, 64, 65, 130])
def test_runs(bias, line, length, moves):
    from paper_2009_09103_amd import csaw
    rp, col = inputs.rmat_csr(11, 4 << 11, 161)  # directed: walks end at sinks
    ew = inputs.rng(162).integers(0, 9, size=len(col)).astype(np.uint32)
    g = csaw.Graph(rp, col, ew)
    for nw in (line - 1, line):
        starts = inputs.walker_starts(rp, col, nw, 163)
        print("[case] runs bias=%d length=%d walkers=%d moves=%s" % (bias, length, nw, moves), flush=True)
        paths, steps = g.walk(starts, length, bias, rng_seed=164, walker_base=7, restart=moves[0], jump=moves[1])
        ids = np.arange(0, nw, 97)
        ref, _, _ = oracle.walk(rp, col, ew, starts[ids], length, bias_kind=bias, rng_seed=164,
                                walker_ids=ids.astype(np.uint64) + 7, restart=moves[0], jump=moves[1])
        got = paths.cpu().numpy()
        np.testing.assert_array_equal(got[ids], ref)
        assert steps == int((got[:, 1:] >= 0).sum())


@pytest.mark.parametrize("moves", [(0, 0), (1 << 29, 1 << 28)])
@pytest.mark.parametrize("bias,line", [(0, 49152), (4, 49152), (1, 45056)])
@pytest.mark.parametrize("length", [1, 33, 65])
def test_runs_from_fewer_walkers(bias, line, length, moves):
    test_runs(bias, line, length, moves)
