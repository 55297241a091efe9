"""The map's counts against its own rays: every binning path of level 3 (the
histogram over a tile's landed-pixel box, the wrapped histogram for boxes
larger than it) must count exactly the pixels that irs_deflect_grid reports
ray by ray."""
import numpy as np
import pytest

import oracle as orc
import synth

pytestmark = pytest.mark.gpu


# pixels from coarse (a tile's box fits the histogram) to far finer than the
# ray spacing (no two rays share a pixel; boxes many wraps wide)
@pytest.mark.parametrize("npix,n_rays,mass", [(16, 150_000, "unit"), (300, 150_001, "unit"),
                                              (1500, 400_003, "salpeter"), (8000, 90_001, "unit")])
def test_counts_equal_binned_pixels(npix, n_rays, mass):
    import torch
    import paper_2204_10871_amd as irs
    kw = dict(kappa_star=0.45, kappa_c=0.05, gamma=0.45, source_side=4.0, npix=npix)
    g = orc.geometry(**kw, n_rays=n_rays)
    L = synth.uniform_lenses(g.n_stars_expected, g.rect, 5, mass=mass)
    p = irs.make_params(**kw, n_rays=n_rays, method="interp", precision="fp64")
    with irs.Plan(p, L.x, L.y, L.m) as pl:
        counts = torch.full((npix * npix,), 7, dtype=torch.int32, device="cuda:0")
        st = pl.shoot_map_device(counts)
        _, _, px = pl.deflect_grid(0, pl.n_rays, alpha=False)
    px = torch.tensor(px[px >= 0], device="cuda:0")
    want = torch.bincount(px, minlength=npix * npix)
    assert st["rays_landed"] == px.numel()
    assert torch.equal(counts.long(), want)
