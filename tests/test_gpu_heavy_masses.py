"""Interpolated deflections scale with the masses up to the ends of the exponent
range: the level-2 series with factorials overflow for masses that the other
forms of the level-2 points still take."""
import numpy as np
import pytest

from gpu_common import Case

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("scale", [2.0 ** 40, 2.0 ** 800])
def test_masses_scale(scale):
    c = Case(kappa_star=0.3, kappa_c=0.0, gamma=0.2, source_side=4.0, npix=32, n_rays=20_000,
             sheet=False)
    c.lenses.m = np.full(c.lenses.n, 1.0)
    n = c.geo.nx * c.geo.ny
    with c.plan("interp", "fp64") as pl:
        a1, a2, _ = pl.deflect_grid(0, n)
        g = pl.geometry
    c.lenses.m = np.full(c.lenses.n, scale)
    with c.plan("interp", "fp64") as pl:
        b1, b2, _ = pl.deflect_grid(0, n)
    # without the macro term the deflections are in proportion to the masses;
    # beside masses of 2^40 and more it is below 1e-11 of them
    i, j = np.arange(n) % g["nx"], np.arange(n) // g["nx"]
    x, y = g["a1"] + (i + 0.5) * g["ray_dx"], g["b1"] + (j + 0.5) * g["ray_dy"]
    a1 = a1 - 0.5 * x
    a2 = a2 - 0.1 * y
    size = np.hypot(a1, a2).max()
    err = np.hypot(b1 / scale - a1, b2 / scale - a2)
    assert np.isfinite(err).all() and err.max() <= 1e-10 * size, err.max()
