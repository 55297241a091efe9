"""FP64 direct sums at the last columns of the ray grid, where a block of 256
columns holds 1 to 255 of them: whole rows of rays against the oracle's direct
definition at the FP64 paths' e_r < 1e-12."""
import numpy as np
import pytest

import oracle as orc
import synth
from gpu_common import Case, THREADS, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("last", [1, 2, 64, 65, 83, 127, 128, 129, 200, 255, 0])
def test_last_columns(last):
    kw = dict(kappa_star=0.3, kappa_c=0.0, gamma=0.3, source_side=4.0, npix=128)
    n_rays = 1 << 20
    while True:                                # the first grid with that many columns past the blocks
        n_rays += 500
        g = orc.geometry(**kw, n_rays=n_rays)
        if g.nx % 256 == last and g.nx * g.ny >= 1 << 20:
            break
    L = synth.uniform_lenses(60, g.rect, 5, mass="salpeter")
    c = Case(**kw, n_rays=n_rays, lenses=L)
    rows = np.array([0, 1, g.ny // 4, g.ny // 2, g.ny - 1])
    ids = (rows[:, None] * g.nx + np.arange(g.nx)).ravel()
    ref = orc.shoot_direct(c.geo, L, ray_ids=ids, want_counts=False, threads=THREADS)
    with c.plan("direct", "fp64") as pl:
        a1, a2, px = pl.deflect_grid(0, pl.n_rays)
        counts, _ = pl.shoot_map()
    e = rel_err(a1[ids], a2[ids], ref["alpha1"], ref["alpha2"])
    assert e.max() < 1e-12, (e.max(), ids[e.argmax()] % g.nx)
    assert np.array_equal(px[ids], ref["pix"])
    assert np.array_equal(np.bincount(px[px >= 0], minlength=128 * 128), counts.ravel())
