"""The routes that the runtime picks for a call, on the host-only build of the
library (tests/hostsim): launchers that note calls given to a kernel that
cannot serve them and read the tables that they are given, under AddressSanitizer + UBSan and under ThreadSanitizer."""
import os
import shutil

import pytest

import test_hostsim as sim

SOURCES = sim.SOURCES[:3] + [os.path.join(sim.SIM, "routes_sim.cpp"), os.path.join(sim.SIM, "routes_driver.cpp")]


@pytest.fixture(scope="module")
def drivers(tmp_path_factory):
    if not shutil.which("g++"):
        pytest.skip("g++ is not available")
    out = str(tmp_path_factory.mktemp("routes"))
    with pytest.MonkeyPatch.context() as patch:
        patch.setattr(sim, "SOURCES", SOURCES)
        return {k: sim.build(k, out) for k in sim.FLAGS}


@pytest.mark.parametrize("scenario", ["replay", "retry", "tables", "room", "give_back", "refused", "autotune", "scratch"])
@pytest.mark.parametrize("kind", ["asan", "tsan"])
def test_routes_under_sanitizers(drivers, kind, scenario):
    sim.run(drivers[kind], scenario)
