"""Layer sampling without a guide at the list lengths where its scan changes: a
quad, a batch of 64 weights and one more, the longest scanned list and the
first that goes through the chunk table, the last list of the weight array
among them; zero weights, weights of 32 bits, few and many rounds. Against the
oracle, element by element."""
import numpy as np
import pytest

import oracle
from paper_2009_09103_amd import inputs

pytestmark = pytest.mark.gpu

LENGTHS = [1, 2, 3, 4, 5, 7, 8, 9, 15, 16, 17, 60, 61, 63, 64, 65, 127, 128, 129, 255, 256, 257, 447, 448, 449, 511, 512, 513]


@pytest.mark.parametrize("last", [1, 3, 64, 65, 512])
@pytest.mark.parametrize("weights", ["plain", "zeros", "wide"])
def test_list_lengths(weights, last):
    from paper_2009_09103_amd import csaw
    gen = inputs.rng(171)
    n = 900
    deg = np.array([LENGTHS[i % len(LENGTHS)] for i in range(n)], dtype=np.int64)
    deg[-1] = last
    rp = np.concatenate([[0], np.cumsum(deg)]).astype(np.int64)
    col = np.concatenate([np.sort(gen.choice(n, size=d, replace=False)) for d in deg]).astype(np.int32)
    col[rp[:-1]] = n - 1 - (np.arange(n) % 2)  # the last lists are picked often
    ew = {"plain": gen.integers(1, 100, size=len(col)), "zeros": gen.integers(0, 9, size=len(col)) * (gen.random(len(col)) < .3),
          "wide": gen.integers((1 << 32) - 99, 1 << 32, size=len(col), dtype=np.uint64)}[weights].astype(np.uint32)
    g = csaw.Graph(rp, col, ew)
    g.set_walk_guides(False)
    sizes = [1, 28, 56, 300]
    seeds = np.concatenate([np.sort(gen.choice(n - 1, size=k - 1, replace=False).tolist() + [n - 1]) for k in sizes]).astype(np.int32)
    offs = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    for kind, rounds in ((1, 0), (1, 1), (2, 0), (1, -1)):
        print("[case] layer lists %s last=%d kind=%d rounds=%d" % (weights, last, kind, rounds), flush=True)
        got = g.layer_sample(offs, seeds, [64, 20, 64], kind, rng_seed=172, rounds=rounds)
        ref = oracle.layer_sample(rp, col, ew, offs, seeds, np.array([64, 20, 64], dtype=np.int32), bias_kind=kind, rng_seed=172,
                                  rounds={0: 8, -1: 0}.get(rounds, rounds))
        for a, b in zip(got, ref):
            np.testing.assert_array_equal(a.cpu().numpy(), b)
