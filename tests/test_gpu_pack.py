"""Packing of the lenses into level-1 cells: one workgroup's sort up to 8192
lenses and 16384 cells, the radix sort beyond.  Whole numbers against numpy's
stable sort of the cell indices; the packed coordinates and masses through the
FP64 direct sum against the same lenses given in packed order."""
import numpy as np
import pytest

import oracle as orc
import synth
from gpu_common import Case, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n,side,where,mass", [
    (1, 2.0, "uniform", "unit"), (2, 2.0, "uniform", "salpeter"), (3, 2.0, "one", "unit"),
    (64, 4.0, "uniform", "unit"), (65, 4.0, "edges", "salpeter"), (127, 4.0, "one", "unit"),
    (1000, 8.0, "clump", "salpeter"), (1024, 8.0, "uniform", "unit"),
    (1025, 8.0, "reverse", "salpeter"), (4097, 8.0, "one", "salpeter"),
    (8191, 20.0, "uniform", "salpeter"), (8192, 20.0, "clump", "unit"),
    (8193, 20.0, "uniform", "unit"),
])
def test_pack_order(n, side, where, mass):
    kw = dict(kappa_star=0.45, kappa_c=0.05, gamma=0.45, source_side=side, npix=16)
    g = orc.geometry(**kw, n_rays=300)
    L = synth.uniform_lenses(n, g.rect, 11, mass=mass)
    a1, a2, b1, b2 = g.rect
    rng = np.random.default_rng(n)
    if where == "one":                         # every lens in one cell
        L.x = 0.3 * a1 + 0.7 * a2 + 1e-3 * rng.random(n)
        L.y = 0.6 * b1 + 0.4 * b2 + 1e-3 * rng.random(n)
    elif where == "clump":
        k = n // 2
        L.x[:k] = a1 + (a2 - a1) * 0.5 + 0.5 * rng.random(k)
        L.y[:k] = b1 + (b2 - b1) * 0.5 + 0.5 * rng.random(k)
    elif where == "edges":                     # on the rectangle's sides and corners
        L.x[::2] = np.where(rng.random(L.x[::2].size) < 0.5, a1, a2)
        L.y[::3] = np.where(rng.random(L.y[::3].size) < 0.5, b1, b2)
    elif where == "reverse":
        o = np.argsort(-L.y, kind="stable")
        L.x, L.y = L.x[o].copy(), L.y[o].copy()
    c = Case(**kw, n_rays=300, lenses=L)
    want_cs, want_perm = orc.level1(c.geo, L)
    with c.plan("direct", "fp64") as pl:
        cs, perm = pl.level1()
        r1, r2, px = pl.deflect_grid(0, pl.n_rays)
    assert np.array_equal(cs, want_cs) and np.array_equal(perm, want_perm)
    L.x, L.y = L.x[perm].copy(), L.y[perm].copy()
    if L.m is not None:
        L.m = L.m[perm].copy()
    with Case(**kw, n_rays=300, lenses=L).plan("direct", "fp64") as pl:
        cs2, perm2 = pl.level1()
        q1, q2, qx = pl.deflect_grid(0, pl.n_rays)
    assert np.array_equal(cs2, cs) and np.array_equal(perm2, np.arange(n))
    # (the masses' sum, and with it the sheet's density, depends on their order)
    assert rel_err(r1, r2, q1, q2).max() < 1e-13 and np.array_equal(px, qx)
