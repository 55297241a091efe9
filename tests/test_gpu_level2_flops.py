"""irs_map_stats.level2_flops counts the work of the level-2 point kernel that
runs: k_level2_cells (the ring lenses once per cell, a quarter of the points
summed) from nine points a cell side on, k_level2_points (every ring lens at
every point) below."""
import numpy as np
import pytest

import synth
from gpu_common import Case

pytestmark = pytest.mark.gpu


def _ring_terms(geo, q):
    """Terms of the cell series with the ring lenses: truncation of c_4 below
    1e-14 at the ratio of the furthest point to the nearest ring lens."""
    w, h = geo.ix / geo.n1x, geo.iy / geo.n1y
    rho = 0.5 * (q - 1) / q * np.hypot(w, h) / (1.5 * min(w, h))
    for P in range(48, 81, 4):
        c4 = P * (P - 1) * (P - 2) * (P - 3) / 24.0
        if c4 * rho ** (P - 4) / (1.0 - rho) ** 5 < 1e-14:
            return P


@pytest.mark.parametrize("q", [20, 9, 8])
def test_level2_points_flops(q):
    kw = dict(kappa_star=0.45, kappa_c=0.05, gamma=0.3, source_side=6.0, npix=64, n_rays=100_000)
    g0 = Case(**kw).geo
    c = Case(**kw, level2_spacing=g0.dx1 / q)
    with c.plan("interp", "fp64") as pl:
        _, st = pl.shoot_map()
        g = pl.geometry
        start, _ = pl.level1()
    assert g["q"] == q
    n1x, n1y = g["n1x"], g["n1y"]
    cells = np.diff(start).reshape(n1y, n1x)

    def block(cy, cx, r):
        return cells[max(0, cy - r):cy + r + 1, max(0, cx - r):cx + r + 1].sum()

    ring = sum(block(cy, cx, 3) - block(cy, cx, 1) for cy in range(n1y) for cx in range(n1x))
    if q >= 9:
        pe, hq = _ring_terms(c.geo, q), (q + 1) // 2
        want = ring * (10 + 8 * pe) + n1x * n1y * (48 * pe * hq * hq + 58 * q * q)
    else:
        want = q * q * (44 * ring + 60 * 32 * n1x * n1y)
    got = st["level2_flops"] - st["level2_expand_flops"]
    assert got == pytest.approx(want, rel=1e-9)
