"""irs_map_stats.ms_total is the call's time on the plan's stream, the copy of a
host map included: on a large map of few rays nearly all of the call's wall
time is that copy, so ms_total has to be most of it."""
import time

import numpy as np
import pytest

import synth
from gpu_common import Case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("call", ["map", "rows"])
def test_ms_total_covers_host_copy(call):
    npix = 8192
    c = Case(kappa_star=0.3, kappa_c=0.0, gamma=0.3, source_side=10.0, npix=npix, n_rays=20_000,
             lenses=synth.Lenses(np.zeros(0), np.zeros(0), None))
    rows = np.zeros((npix, npix), np.uint32)
    with c.plan("direct", "fp64") as pl:
        for _ in range(2):                             # the first call allocates
            t = time.perf_counter()
            st = pl.shoot_map()[1] if call == "map" else pl.shoot_rows(0, c.geo.ny, rows)
            wall = 1e3 * (time.perf_counter() - t)
    assert 0.5 * wall < st["ms_total"] <= wall, (st["ms_total"], wall)
