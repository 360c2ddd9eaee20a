"""Projection of several views with tile culling, as the server asks for it:
together no slower than one view after the other (a thread that takes all views
of its Gaussian waits in each for the lane with the most tiles to test: 1.2
times as long; one thread per record 0.9)."""
import numpy as np
import pytest
import torch

import gs_inputs
from tests import gpu_helpers as H

pytestmark = pytest.mark.gpu


def _ms(f):
    f()
    t = []
    for _ in range(7):
        e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        e0.record()
        f()
        e1.record()
        torch.cuda.synchronize()
        t.append(e0.elapsed_time(e1))
    return float(np.median(t))


def test_culled_views_together(gpu_lib):
    R = H.raster()
    ds = R.DeviceScene.from_numpy(gs_inputs.uniform_cube_scene(1_500_000, 3)).in_spatial_order()[0]
    cams = [gs_inputs.look_at(e, (0, 0, 0), 1280, 720) for e in ((0, 0, 4), (4, 0.5, 0), (2.8, 1, 2.8), (-3, -2, 2))]
    opts, buffers = R.RasterOpts(tile_cull=True), R.StepBuffers()
    alone = sum(_ms(lambda c=c: R.project(ds, [c], opts, buffers=buffers)) for c in cams)
    together = _ms(lambda: R.project(ds, cams, opts, buffers=buffers))
    print(f"together {together:.3f} ms, one after the other {alone:.3f} ms", flush=True)
    assert together < alone
