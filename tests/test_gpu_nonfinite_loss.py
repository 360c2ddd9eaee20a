"""A loss gradient that is NaN or infinite at a few pixels: the 2D gradients it
makes non-finite are those of the Gaussians composited in the 4x4 groups of these
pixels, with the atomics as with the ordered reduction, and no others; all the
rest is what it is without those groups' part."""
import numpy as np
import pytest
import torch

import gs_inputs
from tests import gpu_helpers as H

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("value", [float("nan"), float("inf"), -float("inf")])
@pytest.mark.parametrize("masked", [False, True])
@pytest.mark.parametrize("form", ["whole", "split"])
def test_nonfinite_pixels(gpu_lib, value, masked, form):
    R = H.raster()
    sc = gs_inputs.uniform_cube_scene(3000, 5)
    cam = gs_inputs.look_at((0, 0, 4), (0, 0, 0), 96, 72)
    n, Pn = sc.n, 96 * 72
    ds, opts = R.DeviceScene.from_numpy(sc), R.RasterOpts()
    proj = R.project(ds, [cam], opts)
    binned = R.bin(proj, [cam], n)
    if form == "whole":
        binned.order = None
    frame = R.render_forward(ds, proj, binned, [cam], opts)
    dl = torch.from_numpy(gs_inputs.normal_image(3, Pn, 7, scale=1.0 / Pn)).cuda()
    bad = [(20, 30), (51, 40), (70, 11), (48, 36)]
    for x, y in bad:
        dl[:, y * 96 + x] = value
    mask = torch.from_numpy(gs_inputs.bernoulli_mask(n, 0.5, 3)).cuda() if masked else None
    g = {det: R.render_backward_pixels(proj, binned, [cam], n, opts, frame, dl, mask, deterministic=det)[:n]
         for det in (False, True)}
    odd = {det: ~torch.isfinite(v).all(1) for det, v in g.items()}
    assert 0 < int(odd[True].sum()) < n // 2
    extra = (odd[False] != odd[True]).nonzero()[:, 0]
    assert extra.numel() == 0, (int(odd[False].sum()), int(odd[True].sum()), extra[:8].tolist())
    a, b = g[False][~odd[True]].double(), g[True][~odd[True]].double()
    assert float((a - b).norm() / b.norm()) < 1e-5
