"""Level 3's waves of ray rows: they follow the level-1 cells' rows wherever
every cell has one (from one row a cell up, with rows to spare at a cell's end)
and are cut every eight rows otherwise.  Against the oracle's interpolation
(e_r < 1e-10, the FP64 path's tolerance), the map against the rays' own pixels,
and any range of rays with the bits of the whole grid."""
import numpy as np
import pytest

import oracle as orc
import synth
from gpu_common import Case, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("rows,mass", [(0.6, "unit"), (1.3, "unit"), (3.5, "salpeter"),
                                       (8.0, "unit"), (9.1, "unit"), (17.0, "salpeter"),
                                       (33.2, "unit")])
def test_ray_rows(rows, mass):
    kw = dict(kappa_star=0.45, kappa_c=0.05, gamma=0.2, source_side=12.0, npix=48)
    g = orc.geometry(**kw, n_rays=1000)
    cells = orc.geometry(**kw, n_rays=1000).with_lens_count(g.n_stars_expected)
    n_rays = int(rows ** 2 * cells.n1x * cells.n1y)
    L = synth.uniform_lenses(g.n_stars_expected, g.rect, 7, mass=mass)
    c = Case(**kw, n_rays=n_rays, lenses=L)
    ref = c.oracle_interp()
    with c.plan("interp", "fp64") as pl:
        nx, ny, n = pl.geometry["nx"], pl.geometry["ny"], pl.n_rays
        assert abs(ny / pl.geometry["n1y"] - rows) < 0.15 * rows + 0.1
        a1, a2, px = pl.deflect_grid(0, n)
        counts, st = pl.shoot_map()
        for j0, j1 in ((0, 1), (ny - 1, ny), (ny // 2 - 3, ny // 2 + 8), (5, min(ny, 38))):
            f, l = max(0, j0) * nx + (j1 - j0 > 1) * (nx // 3), min(ny, j1) * nx
            b1, b2, bx = pl.deflect_grid(f, l - f)
            assert np.array_equal(a1[f:l], b1) and np.array_equal(a2[f:l], b2) and \
                np.array_equal(px[f:l], bx)
    assert rel_err(a1, a2, ref["alpha1"], ref["alpha2"]).max() < 1e-10
    assert np.mean(px == ref["pix"]) >= 1 - 1e-5
    assert st["rays_landed"] == (px >= 0).sum()
    assert np.array_equal(np.bincount(px[px >= 0], minlength=48 * 48), counts.ravel())


@pytest.mark.parametrize("mass", ["unit", "salpeter"])
def test_half_waves(mass):
    """A call of few rays takes waves of four rows, the whole grid (5740 waves of
    eight) does not: the same bits, the map's counts the rays' pixels."""
    kw = dict(kappa_star=0.45, kappa_c=0.05, gamma=0.2, source_side=12.0, npix=256)
    g = orc.geometry(**kw, n_rays=2_960_000)
    c = Case(**kw, n_rays=2_960_000, lenses=synth.uniform_lenses(g.n_stars_expected, g.rect, 7,
                                                                 mass=mass))
    with c.plan("interp", "fp64") as pl:
        nx, ny, n = pl.geometry["nx"], pl.geometry["ny"], pl.n_rays
        a1, a2, px = pl.deflect_grid(0, n)
        counts, _ = pl.shoot_map()
        for f, l in ((0, 3), (n - 700, n), (81 * nx - 5, 81 * nx + 5), (ny // 2 * nx + 11, ny // 2 * nx + 9 * nx),
                     (7 * nx, 8 * nx), (300 * nx + nx // 2, 340 * nx)):
            b1, b2, bx = pl.deflect_grid(f, l - f)
            assert np.array_equal(a1[f:l], b1) and np.array_equal(a2[f:l], b2) and \
                np.array_equal(px[f:l], bx), (f, l)
    assert np.array_equal(np.bincount(px[px >= 0], minlength=256 * 256), counts.ravel())
