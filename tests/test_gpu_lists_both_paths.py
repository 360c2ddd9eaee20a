"""Both ways to the tile lists, each where it is the subject: the radix sort of
(tile | depth) keys through gs_bin_count and gs_bin_sort, and the lists by tile
through gs_bin (max_list > 0 says that they were made so), against the oracle's
binning and against each other."""
import numpy as np
import pytest
import torch

import gs_inputs
import oracle
from tests import gpu_helpers as H
from tests.test_gpu_parity import count_path  # noqa: F401 - a fixture
from tests.test_gpu_tile_lists import DEPTHS, _Cam, _compare, _projected

pytestmark = pytest.mark.gpu


def _np(t):
    return t.detach().cpu().numpy()


def _views(seed, n):
    sc = gs_inputs.uniform_cube_scene(n, seed)
    return sc, [gs_inputs.look_at((0, 0, 4), (0, 0, 0), 128, 128), gs_inputs.look_at((2.5, 1, 3), (0, 0, 0), 150, 77)]


def _check(b, sc, cams, what):
    p, rects, zb = oracle.Params.of(sc), [], []
    for cam in cams:
        P = oracle.project(p, cam, oracle.Opts())
        rects.append(oracle.tile_rects(P))
        zb.append(oracle.zbits(P))
    rects, zb = np.concatenate(rects), np.concatenate(zb)
    tx, _, base, total = oracle.view_layout(cams)
    keys, vals, ranges = oracle.bin(rects, zb, len(cams), sc.n, base, tx, total)
    torch.cuda.synchronize()
    assert b.stats.n_isect == len(keys), what
    assert np.array_equal(_np(b.keys).view(np.uint64), keys), what
    assert np.array_equal(_np(b.vals).view(np.uint32), vals), what
    assert np.array_equal(_np(b.ranges).view(np.uint32), ranges), what
    H.check_bin_extras(b, rects, zb, len(cams), total, ranges, what)


@pytest.mark.parametrize("views", [1, 2])
def test_radix_sort_against_the_oracle(gpu_lib, count_path, views):  # noqa: F811
    R = H.raster()
    sc, cams = _views(1, 4096)
    cams = cams[:views]
    proj = R.project(R.DeviceScene.from_numpy(sc), cams, R.RasterOpts())
    offsets, st = R.bin_count(proj, cams, sc.n)
    assert st.max_list == 0
    _check(R.bin_sort(proj, cams, sc.n, offsets, st, want_keys=True), sc, cams, f"radix, {count_path}, {views} views")


@pytest.mark.parametrize("views", [1, 2])
def test_lists_by_tile_against_the_oracle(gpu_lib, views):
    R = H.raster()
    sc, cams = _views(1, 4096)
    cams = cams[:views]
    proj = R.project(R.DeviceScene.from_numpy(sc), cams, R.RasterOpts())
    b = R.bin(proj, cams, sc.n, want_keys=True)
    assert b.stats.max_list > 0
    _check(b, sc, cams, f"by tile, {views} views")


def test_one_call_equals_count_and_sort(gpu_lib):
    """gs_bin into growing and into larger buffers against the separate calls."""
    R = H.raster()
    bufs = R.StepBuffers()
    for seed, n in ((21, 4096), (21, 4096), (22, 9000), (23, 1000), (24, 0)):
        sc, cams = _views(seed, max(n, 1))
        if n == 0:
            sc.opacity[:] = 0.0  # nothing reaches alpha_min: no pairs
        proj = R.project(R.DeviceScene.from_numpy(sc), cams, R.RasterOpts())
        one = R.bin_step(proj, cams, sc.n, bufs, want_keys=True)
        offsets, st = R.bin_count(proj, cams, sc.n)
        two = R.bin_sort(proj, cams, sc.n, offsets, st, want_keys=True)
        torch.cuda.synchronize()
        assert (one.stats.max_list > 0) == (n > 0) and st.n_isect == one.stats.n_isect
        for f in ("keys", "vals", "ranges", "order", "offsets"):
            assert torch.equal(getattr(one, f), getattr(two, f)), (n, f)


@pytest.mark.parametrize("n,sizes", [(300, [(17, 16)]), (257, [(2100, 1100), (33, 700)]),
                                     (5000, [(640, 480), (64, 48), (801, 603)])])
def test_boxes_of_all_sizes_by_tile(gpu_lib, n, sizes):
    """Boxes from one pixel to the whole image in records sorted by place, some
    not drawn: all by tile."""
    R = H.raster()
    g = gs_inputs.rng(n)
    cams, boxes = [_Cam(w, h) for w, h in sizes], []
    for w, h in sizes:
        x, y = g.integers(0, w, n), g.integers(0, h, n)
        o = np.lexsort((x // 64, y // 64))
        x, y = x[o], y[o]
        half = np.where(g.uniform(size=n) < 0.02, 4096, g.integers(0, 24, n))
        b = np.stack([np.maximum(x - half, 0), np.minimum(x + half, w - 1), np.maximum(y - half, 0),
                      np.minimum(y + half, h - 1)], 1)
        b[g.uniform(size=n) < 0.2] = (1, 0, 1, 0)
        boxes.append(b)
    z = np.concatenate([DEPTHS["spread"](g, n) for _ in sizes])
    assert _compare(R, _projected(R, cams, np.concatenate(boxes), z), cams, n, f"n={n} {sizes}").max_list > 0


@pytest.mark.parametrize("cull", [False, True])
def test_projected_scene_by_tile(gpu_lib, cull):
    R = H.raster()
    sc, cams = _views(4, 6000)
    proj = R.project(R.DeviceScene.from_numpy(sc), cams, R.RasterOpts(tile_cull=cull))
    assert _compare(R, proj, cams, sc.n, f"cull {cull}").max_list > 0
