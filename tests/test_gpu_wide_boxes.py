"""Boxes of thousands of tiles, whose workgroups count and place in bands of
tile rows: the lists against the radix sort, bitwise, with and without tile
culling, and the walk's cost, which must not grow with the number of bands."""
import numpy as np
import pytest
import torch

import gs_inputs
from tests import gpu_helpers as H
from tests.test_gpu_tile_lists import _compare

pytestmark = pytest.mark.gpu


def _scene(n, wide, seed=0, scale=3.0):
    """n small Gaussians and `wide` that reach over the whole view."""
    g = gs_inputs.rng(seed)
    sc = gs_inputs.uniform_cube_scene(n + wide, seed)
    sc.means[:, n:] = 0.3 * g.normal(size=(3, wide))
    sc.scales[:, :n] *= 0.2
    sc.scales[:, n:] = scale
    sc.opacity[n:] = 0.05
    return sc


def _records(R, sc, cams, cull):
    ds = R.DeviceScene.from_numpy(sc).in_spatial_order()[0]
    return R.project(ds, cams, R.RasterOpts(tile_cull=cull)), ds.n


@pytest.mark.parametrize("cull", [False, True])
@pytest.mark.parametrize("size", [(1024, 512), (1040, 528), (1920, 1080), (4096, 330), (330, 4096)])
def test_lists_in_bands(gpu_lib, size, cull):
    R = H.raster()
    cams = [gs_inputs.look_at((0, 0, 4), (0, 0, 0), *size)]
    sc = _scene(3000, 100)
    if cull:  # tilted needles of a few tiles among them, which lose some
        sc.scales[0, 2000:3000], sc.scales[1:, 2000:3000] = 0.08, 0.005
    proj, n = _records(R, sc, cams, cull)
    if cull:
        b = proj.bin.cpu().numpy().view(np.uint32)[:n].astype(np.int64)
        boxes = ((b[:, 0] >> 20) - ((b[:, 0] & 0xffff) >> 4) + 1) * ((b[:, 1] >> 20) - ((b[:, 1] & 0xffff) >> 4) + 1)
        assert ((b[:, 3] > 0) & (b[:, 3] < boxes)).sum() > 100
    st = _compare(R, proj, cams, n, f"{size} cull {cull}")
    assert st.max_list > 0


def test_cost_does_not_grow_with_the_bands(gpu_lib):
    """3840x2160: 17 bands.  A pair walked once per kernel and pass costs a
    fraction of the radix sort's passes; walked once per band it costs as much
    as all of it (8.7 against 8.5 ms; now 1.1)."""
    R = H.raster()
    cams = [gs_inputs.look_at((0, 0, 4), (0, 0, 0), 3840, 2160)]
    proj, n = _records(R, _scene(200_000, 512), cams, False)
    by_tile, radix = R.StepBuffers(), R.BinBuffers()

    def lists():
        return R.bin_step(proj, cams, n, by_tile)

    def sorted_lists():
        offsets, st = R.bin_count(proj, cams, n)
        return R.bin_sort(proj, cams, n, offsets, st, buffers=radix)

    def ms(f):
        f()
        t = []
        for _ in range(5):
            e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            e0.record()
            f()
            e1.record()
            torch.cuda.synchronize()
            t.append(e0.elapsed_time(e1))
        return float(np.median(t))

    assert lists().stats.max_list > 0
    a, b = ms(lists), ms(sorted_lists)
    print(f"by tile {a:.2f} ms, radix {b:.2f} ms", flush=True)
    assert a < 0.5 * b


def _tiles(R, cam, boxes):
    """gs_bin_tiles alone of one view's boxes: the statistics."""
    import ctypes
    from paper_2411_12788_amd import _lib as L
    from tests.test_gpu_tile_lists import _projected
    n, tiles, lib = len(boxes), R.tiles_total([cam]), L.lib()
    proj = _projected(R, [cam], boxes, np.linspace(1.0, 2.0, n))
    offsets = torch.empty(n, dtype=torch.int32, device="cuda")
    ranges = torch.empty(2 * tiles, dtype=torch.int32, device="cuda")
    order = torch.empty(tiles, dtype=torch.int32, device="cuda")
    ws = torch.empty(lib.gs_bin_count_workspace_size(n), dtype=torch.uint8, device="cuda")
    st, pc = L.BinStats(), proj.c()
    L.check(lib.gs_bin_tiles(ctypes.byref(pc), R.cameras([cam]), 1, n, R._ptr(offsets), ctypes.byref(st),
                             R._ptr(ranges), R._ptr(order), R._ptr(ws), ws.numel(), R._stream()), "gs_bin_tiles")
    torch.cuda.synchronize()
    return st


@pytest.mark.parametrize("side,n,by_tile", [
    (1024, 128, True),    # half of a workgroup's records as large as the largest
    (1024, 129, False),   # more: one workgroup would do all the work
    (1024, 513, False),
    (256, 256, True),     # few pairs: no matter
    (8192, 256, False),   # 2^26 pairs in the one group, sampled 64 times: 2^32 in all
])
def test_groups_of_boxes_as_large_as_the_view(gpu_lib, side, n, by_tile):
    from tests.test_gpu_tile_lists import _Cam
    R = H.raster()
    st = _tiles(R, _Cam(side, side), [(0, side - 1, 0, side - 1)] * n)
    assert st.n_isect == n * (side // 16) ** 2
    assert st.max_list == (n if by_tile else 0)
