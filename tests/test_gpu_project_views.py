"""Projection of several views at once around the size from which a thread
takes all views of its Gaussian, against one call per view: pixel boxes, tile
counts and depths equal, records equal to the rounding of float32 (both round
the same double expressions, which the compiler may fuse differently), for
every SH degree, with a culling mask, zero quaternions, Gaussians behind a
camera and non-finite coefficients."""
import numpy as np
import pytest
import torch

import gs_inputs
from tests import gpu_helpers as H

pytestmark = pytest.mark.gpu

EDGE = 1 << 16


@pytest.mark.parametrize("degree", [0, 1, 2, 3])
@pytest.mark.parametrize("n,V", [(EDGE - 1, 2), (EDGE, 2), (EDGE + 17, 3), (EDGE + 255, 16)])
@pytest.mark.parametrize("tile_cull", [False, True])
def test_views_together_equal_views_alone(gpu_lib, degree, n, V, tile_cull):
    R = H.raster()
    sc = gs_inputs.uniform_cube_scene(n, 5)
    g = gs_inputs.rng(6)
    sc.sh_degree = degree
    sc.quats[:, g.integers(0, n, 50)] = 0.0
    sc.sh[0, 1, g.integers(0, n, 20)] = np.nan
    mask = torch.from_numpy((g.random(n) < 0.9).astype(np.uint8)).cuda()
    # cameras inside and outside the cube: some Gaussians lie behind them
    cams = [gs_inputs.look_at((0.2 * k, 0.1, 0.3 + 1.1 * (k % 4)), (0.0, 0.0, -0.2), 160 + 16 * k, 120)
            for k in range(V)]
    ds = R.DeviceScene.from_numpy(sc)
    opts = R.RasterOpts(tile_cull=tile_cull)
    print(f"n={n}, V={V}, degree={degree}, tile_cull={tile_cull}", flush=True)
    both = R.project(ds, cams, opts, mask)
    torch.cuda.synchronize()
    drawn = 0
    for v, cam in enumerate(cams):
        one = R.project(ds, [cam], opts, mask)
        torch.cuda.synchronize()
        rows = slice(v * n, (v + 1) * n)
        assert torch.equal(both.bin[rows], one.bin)
        keep = one.bin[:, 3] > 0
        drawn += int(keep.sum())
        a, b = both.rec[rows][keep].double(), one.rec[keep].double()
        # the mean is held as a pair: high part and what it leaves
        for c in (0, 1):
            pa, pb = a[:, c] + a[:, c + 2], b[:, c] + b[:, c + 2]
            assert ((pa - pb).abs() <= 2.0 ** -44 * pb.abs().clamp(min=1.0)).all()
        rest = [4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15]
        scale = b[:, rest].abs()
        scale[:, [1, 9]] = torch.maximum(scale[:, [1, 9]], scale[:, [0, 8]])  # the cross term may cancel
        scale[:, [4, 5, 6]] = scale[:, [4, 5, 6]].clamp(min=1.0)  # so may a colour's terms
        assert ((a[:, rest] - b[:, rest]).abs() <= 2.0 ** -23 * scale).all()
    assert drawn > n // 4
