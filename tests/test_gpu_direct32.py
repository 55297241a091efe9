"""The FP32 direct sum's cut of a call's rays into one piece per wave: each ray
is summed with the same operations wherever the cut lies, so deflections and
pixels are the same bits in any range they are asked for, in every tile shape,
and within the FP32 path's tolerance (e_r <= 1e-5) of the FP64 sum."""
import numpy as np
import pytest

import oracle as orc
import synth
from gpu_common import Case, rel_err

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_rays,gamma,n_lens,mass", [
    (1, 0.45, 3, "unit"),
    (64 * 65, -0.45, 31, "salpeter"),       # few columns, rows of one piece each
    (20_011, 0.45, 33, "unit"),
    (300_007, 0.3, 257, "salpeter"),        # more than one stage of lenses
    (1_000_003, 0.0, 40, "unit"),           # more than one round of pieces at 4 rows a lane
])
def test_direct32_pieces(n_rays, gamma, n_lens, mass):
    kw = dict(kappa_star=0.45, kappa_c=0.05, gamma=gamma, source_side=2.0, npix=64)
    g = orc.geometry(**kw, n_rays=n_rays)
    c = Case(**kw, n_rays=n_rays, lenses=synth.uniform_lenses(n_lens, g.rect, 3, mass=mass))
    with c.plan("direct", "fp32") as pl, c.plan("direct", "fp64") as p64:
        nx, ny, n = pl.geometry["nx"], pl.geometry["ny"], pl.n_rays
        pl.set_direct_variant(0)
        a1, a2, px = pl.deflect_grid(0, n)
        for v in (1, 2):
            pl.set_direct_variant(v)
            b1, b2, bx = pl.deflect_grid(0, n)
            assert np.array_equal(a1, b1) and np.array_equal(a2, b2) and np.array_equal(px, bx)
        r1, r2, _ = p64.deflect_grid(0, n)
        pl.set_direct_variant(1)
        counts, st = pl.shoot_map()
        assert np.array_equal(np.bincount(px[px >= 0], minlength=64 * 64), counts.ravel())
        assert st["rays_landed"] == (px >= 0).sum()
        rows = [(0, 1), (ny - 1, ny), (ny // 2, ny // 2 + 9)]
        spans = [(max(0, r0) * nx, min(ny, r1) * nx) for r0, r1 in rows]
        mid = ny // 3 * nx
        spans += [(0, 1), (n - 1, n), (mid + nx // 2, mid + nx // 2 + 1),
                  (mid + nx - 1, min(n, mid + nx + 1)), (min(mid + 3, n - 1), min(n, mid + 5 * nx))]
        for f, l in spans:
            b1, b2, bx = pl.deflect_grid(f, l - f)
            assert np.array_equal(a1[f:l], b1) and np.array_equal(a2[f:l], b2) and \
                np.array_equal(px[f:l], bx), (f, l)
    assert rel_err(a1, a2, r1, r2).max() <= 1e-5
