"""The FP64 direct sum's forms against the oracle's direct definition: four rays
a lane (calls of 2^20 rays or more) and one, waves inside one ray row and across
rows, lenses exactly on rays and on ray rows, masses that switch the refined
reciprocals off.  Tolerance: the FP64 paths' e_r < 1e-12."""
import numpy as np
import pytest

import oracle as orc
import synth
from gpu_common import Case, THREADS, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("gamma,n_rays,mass", [
    (0.45, (1 << 20) + 77, "unit"),        # four a lane, rows of thousands of rays
    (-0.45, (1 << 20) + 5, "salpeter"),    # ... rows shorter than a wave's 256 rays
    (0.45, 300_007, "salpeter"),           # one a lane
    (0.45, 1_200_003, "heavy"),            # a mass outside the refined reciprocals' range
    (0.45, 1_200_003, "on_rays"),
])
def test_direct64_forms(gamma, n_rays, mass):
    kw = dict(kappa_star=0.45, kappa_c=0.05, gamma=gamma, source_side=2.0, npix=64)
    g = orc.geometry(**kw, n_rays=n_rays)
    L = synth.uniform_lenses(g.n_stars_expected, g.rect, 3,
                             mass="salpeter" if mass == "salpeter" else "unit")
    g = g.with_lens_count(L.n)
    if mass == "heavy":
        L.m = np.ones(L.n)
        L.m[5] = 1e-101
    rng = np.random.default_rng(2)
    near = []
    if mass == "on_rays":
        for k in range(12):                # on a ray, or on a ray row between rays
            i, j = int(rng.integers(g.nx)), int(rng.integers(g.ny))
            L.x[k] = g.a1 + (i + (0.5 if k % 2 else 0.75)) * g.ray_dx
            L.y[k] = g.b1 + (j + 0.5) * g.ray_dy
            near += [j * g.nx + ii for ii in range(max(0, i - 300), min(g.nx, i + 300))]
    ids = np.unique(np.concatenate([rng.integers(0, g.nx * g.ny, 2000), np.arange(700),
                                    g.nx * g.ny - 1 - np.arange(700),
                                    np.array(near, np.int64)]))
    c = Case(**kw, n_rays=n_rays, lenses=L)
    ref = orc.shoot_direct(c.geo, L, ray_ids=ids, want_counts=False, threads=THREADS)
    with c.plan("direct", "fp64") as pl:
        a1, a2, px = pl.deflect_grid(0, pl.n_rays)
        counts, st = pl.shoot_map()
        b1, b2, bx = pl.deflect_grid(1001, 60_000)           # one a lane, unaligned
    e = rel_err(a1[ids], a2[ids], ref["alpha1"], ref["alpha2"])
    assert e.max() < 1e-12, e.max()
    assert np.array_equal(px[ids], ref["pix"])
    assert np.array_equal(np.bincount(px[px >= 0], minlength=64 * 64), counts.ravel())
    s = slice(1001, 61_001)
    assert rel_err(a1[s], a2[s], b1, b2).max() < 1e-14 and np.array_equal(px[s], bx)
