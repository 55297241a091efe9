"""The FP64 direct map's sheet along ray rows (a series about the middle of a
wave's 256 rays, the closed form near the rectangle's corners) against the
closed form that the per-ray deflections take: on pixels of 1e-3 and less no
ray may change its pixel (an error of 1e-9 would move about a hundred)."""
import numpy as np
import pytest

import oracle as orc
import synth
from gpu_common import Case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("gamma,side,npix,n_rays", [
    (0.45, 2.0, 4000, (1 << 20) + 1),        # long rows: most waves take the series
    (0.0, 4.0, 4000, (1 << 20) + 1),         # 1024 rays a row: a quarter of it a wave
    (0.2, 30.0, 8000, 2_000_003),
    (-0.3, 3.0, 3000, (1 << 20) + 1),        # rows shorter than columns
])
def test_sheet_rows(gamma, side, npix, n_rays):
    kw = dict(kappa_star=0.4, kappa_c=0.1, gamma=gamma, source_side=side, npix=npix)
    g = orc.geometry(**kw, n_rays=n_rays)
    c = Case(**kw, n_rays=n_rays, lenses=synth.uniform_lenses(40, g.rect, 4, mass="salpeter"))
    with c.plan("direct", "fp64") as pl:
        _, _, px = pl.deflect_grid(0, pl.n_rays, alpha=False)
        counts, st = pl.shoot_map()
    assert st["rays_landed"] == (px >= 0).sum()
    assert np.array_equal(np.bincount(px[px >= 0], minlength=npix * npix), counts.ravel())
