"""Which profile scopes time a sampling call's selection, and the bytes that
bench.py gives them: weighted lists before their guide, with and without lanes
that scan short ones, and with the guide."""
import importlib.util
import os

import pytest

from paper_2009_09103_amd import inputs

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SCOPES = ("select_slots", "select_wave", "select_big")


@pytest.fixture(scope="module")
def bench():
    spec = importlib.util.spec_from_file_location("bench_scopes", os.path.join(ROOT, "bench.py"))
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod


ALG = {"select_small": 1.0, "select_wave": 10.0, "select_big": 100.0}


@pytest.mark.parametrize("launches,want,main", [
    ((3, 0, 0), {"select_slots": 111.0}, "select_slots"),
    ((3, 0, 3), {"select_slots": 1.0, "select_big": 110.0}, "select_slots"),
    ((0, 3, 3), {"select_wave": 11.0, "select_big": 100.0}, "select_wave"),
])
def test_bytes_go_to_the_scope_that_moves_them(bench, launches, want, main):
    assert bench.select_bytes(ALG, dict(zip(SCOPES, ((0.1 * n, n) for n in launches)))) == (want, main)
    assert set(want) <= set(bench.SELECT_SCOPES)


@pytest.mark.gpu
def test_scopes_name_their_kernels():
    from paper_2009_09103_amd import csaw
    rp, col = inputs.rmat_csr(13, 16 << 13, 141)
    offs, seeds = inputs.single_instance_seeds(rp, col, 300, 142)
    g = csaw.Graph(rp, col)

    def scopes():
        csaw.profile_reset()
        csaw.profile_enable(True)
        g.sample(offs, seeds, [10, 5], csaw.NEIGHBOR_DEGREE, rng_seed=143)
        csaw.profile_enable(False)
        got = {k: csaw.profile_read(k) for k in SCOPES}
        csaw.profile_reset()
        assert all((ms > 0) == (n > 0) for ms, n in got.values()), got
        return {k: n for k, (_, n) in got.items() if n}

    print("[case] scopes", flush=True)
    assert scopes() == {"select_slots": 2, "select_big": 2}
    g.set_tuning(0, 0)
    assert scopes() == {"select_wave": 2, "select_big": 2}
    g.walk(seeds[:1], 1, csaw.NEIGHBOR_DEGREE)  # builds the guide
    assert scopes() == {"select_slots": 2}
