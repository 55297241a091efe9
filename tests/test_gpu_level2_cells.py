"""The level-2 points from one expansion per cell with its ring lenses, at
coarse grids around the sizes where the kernel changes form (below 9 points a
cell side the ring lenses are summed at every point; even and odd sides; one and
several passes of a wave over a cell's quarter), against the oracle's
interpolation (which sums every distant lens at every point): e_r < 1e-10."""
import numpy as np
import pytest

import oracle as orc
import synth
from gpu_common import Case, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("q,mass,clump", [(8, "unit", 0), (9, "salpeter", 0), (13, "unit", 0),
                                          (16, "unit", 60), (20, "salpeter", 0), (27, "unit", 0)])
def test_level2_cells(q, mass, clump):
    kw = dict(kappa_star=0.4, kappa_c=0.0, gamma=0.3, source_side=3.0, npix=64)
    g = orc.geometry(**kw, n_rays=60_001)
    L = synth.uniform_lenses(g.n_stars_expected, g.rect, 8, mass=mass)
    if clump:                                  # lenses crowded into one spot, others empty
        L.x[:clump] = 0.3 + 0.02 * np.arange(clump) / clump
        L.y[:clump] = -0.4 + 0.03 * np.cos(np.arange(clump))
    dx1 = g.with_lens_count(L.n).dx1
    c = Case(**kw, n_rays=60_001, lenses=L, level2_spacing=dx1 / q)
    assert c.geo.q == q
    ref = c.oracle_interp()
    with c.plan("interp") as pl:
        assert pl.geometry["q"] == q
        a1, a2, px = pl.deflect_grid(0, pl.n_rays)
    e = rel_err(a1, a2, ref["alpha1"], ref["alpha2"])
    assert e.max() < 1e-10, e.max()
    assert np.mean(px == ref["pix"]) >= 0.9999
