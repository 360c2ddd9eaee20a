"""Lists around the lengths of the compositing kernels' rounds (192 and 256
staged entries) and chunks (64): one tile that holds every Gaussian, as a whole
work item, as split ones, and as the one tile with entries among empty ones
(the forward then composites four entries side by side).  Forward outputs and
accumulations against the oracle, gradients of the masked, unmasked and
deterministic kernels by relative L2."""
import dataclasses

import numpy as np
import pytest
import torch

import gs_inputs
import oracle
from tests import gpu_helpers as H

pytestmark = pytest.mark.gpu

LENGTHS = (1, 2, 63, 64, 65, 129, 191, 192, 193, 255, 256, 257, 385, 513)


def _np(t):
    return t.detach().cpu().numpy()


@pytest.mark.parametrize("n", LENGTHS)
@pytest.mark.parametrize("form", ["whole", "split", "alone"])
def test_list_lengths_around_rounds(gpu_lib, n, form):
    R = H.raster()
    # "alone": nine tiles, every Gaussian inside the middle one
    wl = (gs_inputs.heavy_tiles(seed=11 + n, n=n, width=48, height=48, opacity=(0.05, 0.6), distance=12.0)
          if form == "alone" else
          gs_inputs.heavy_tiles(seed=11 + n, n=n, width=16, height=16, opacity=(0.01, 0.1), distance=4.0))
    cam = wl.cameras[0]
    Pn = cam.width * cam.height
    print(f"list of {n}, {form}", flush=True)
    ds = R.DeviceScene.from_numpy(wl.scene)
    opts = R.RasterOpts()
    proj = R.project(ds, wl.cameras, opts)
    binned = R.bin(proj, wl.cameras, n)
    rng = _np(binned.ranges).reshape(-1, 2)
    lens = rng[:, 1] - rng[:, 0]
    assert lens.max() == lens.sum() == n  # one tile holds them all
    if form == "whole":
        binned = dataclasses.replace(binned, order=None)
    acc = R.alloc_accum(n, 1, False)
    frame = R.render_forward(ds, proj, binned, wl.cameras, opts, accum=acc)
    p = oracle.Params.of(wl.scene)
    orc = oracle.forward_view(p, cam, oracle.Opts())
    flips, _ = H.compare_forward(frame, orc, slice(0, Pn), f"list of {n}, {form}", p, cam)
    H.check_accum(acc, p, cam, orc["proj"], orc["order"], oracle.Opts(), flips, n, f"list of {n}, {form}")
    dldc = gs_inputs.normal_image(3, Pn, 61, scale=1.0 / Pn)
    for mask in (None, gs_inputs.bernoulli_mask(n, 0.25, 62)):
        og, og2d = H.backward_views(p, wl.cameras, oracle.Opts(), [dldc.T.astype(np.float64)], active=mask,
                                    flips=[flips])
        want = og2d[0] if mask is None else og2d[0] * mask[:, None]
        for det in (False, True):
            grads, g2d = R.render_backward(ds, proj, binned, wl.cameras, opts, frame, torch.from_numpy(dldc).cuda(),
                                           None if mask is None else torch.from_numpy(mask).cuda(), deterministic=det)
            torch.cuda.synchronize()
            got = _np(g2d).astype(np.float64)[:n]
            if not want.any():
                assert not got.any()
                continue
            assert H.rel_l2(got, want) <= H.GRAD_REL_L2, (mask is None, det)
            for k in ("means", "scales", "quats", "opacity", "sh"):
                assert H.rel_l2(_np(grads[k])[..., :n].astype(np.float64), og[k]) <= H.GRAD_REL_L2, (k, det)
