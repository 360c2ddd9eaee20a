"""Tile lists made by tile (gs_bin_tiles, gs_bin_lists) against the radix sort
of (tile | depth) keys (gs_bin_count, gs_bin_sort), bitwise: values, keys,
ranges, tile order and offsets, at the edges of the workgroup sort (lists of one,
512, 2,048 and 8,192 entries and one more, slices of long lists, the limit above which the radix
sort takes over), with equal and bunched depths, culled tiles, several views
and boxes of one tile up to the whole image."""
import ctypes

import numpy as np
import pytest
import torch

import gs_inputs
from tests import gpu_helpers as H

pytestmark = pytest.mark.gpu


class _Cam:
    """Sizes are all that the binning reads of a camera."""

    def __init__(self, w, h):
        self.R, self.t = np.eye(3, dtype=np.float32), np.zeros(3, dtype=np.float32)
        self.fx = self.fy = 100.0
        self.cx, self.cy, self.width, self.height = w / 2, h / 2, w, h


def _projected(R, cams, boxes, z):
    """Records [V * n] with the given pixel boxes (x0, x1, y0, y1; x1 < x0: not
    drawn) and depths; conics and colours are not read without tile culling."""
    boxes = np.asarray(boxes, dtype=np.int64)
    b = np.zeros((len(boxes), 4), dtype=np.uint32)
    b[:, 0] = (boxes[:, 0] & 0xFFFF) | ((boxes[:, 1] & 0xFFFF) << 16)
    b[:, 1] = (boxes[:, 2] & 0xFFFF) | ((boxes[:, 3] & 0xFFFF) << 16)
    b[:, 2] = np.asarray(z, dtype=np.float32).view(np.uint32)
    drawn = boxes[:, 1] >= boxes[:, 0]
    tiles = ((boxes[:, 1] >> 4) - (boxes[:, 0] >> 4) + 1) * ((boxes[:, 3] >> 4) - (boxes[:, 2] >> 4) + 1)
    b[:, 3] = np.where(drawn, tiles, 0)
    rec = torch.zeros((len(boxes), 16), device="cuda")
    return R.Projected(rec, torch.from_numpy(b.view(np.int32)).cuda())


def _compare(R, proj, cams, n, what):
    got = R.bin(proj, cams, n, want_keys=True)
    offsets, st = R.bin_count(proj, cams, n)
    ref = R.bin_sort(proj, cams, n, offsets, st, want_keys=True)
    torch.cuda.synchronize()
    print(what, "pairs", st.n_isect, "longest", got.stats.max_list, "slices", got.stats.list_slices, flush=True)
    for f in ("n_isect", "n_visible", "zbits_min", "zbits_max", "tiles_total", "depth_bits", "key_bits"):
        assert getattr(got.stats, f) == getattr(st, f), f
    assert torch.equal(got.offsets, ref.offsets)
    assert torch.equal(got.ranges, ref.ranges)
    assert torch.equal(got.keys, ref.keys)
    assert torch.equal(got.vals, ref.vals)
    assert torch.equal(got.order, ref.order)
    lengths = (ref.ranges[:, 1] - ref.ranges[:, 0]).cpu().numpy()
    assert got.stats.max_list in (0, lengths.max())
    return got.stats


DEPTHS = {
    "spread": lambda g, m: g.uniform(0.5, 40.0, m),
    "equal": lambda g, m: np.full(m, 3.25),
    # one near Gaussian stretches the range, the rest in a few thousand float steps
    "bunched": lambda g, m: np.where(np.arange(m) == m // 2, 0.2, 30.0 + g.integers(0, 4000, m) * 1.9e-6),
    "few values": lambda g, m: 2.0 + g.integers(0, 3, m) * 0.25,
}


@pytest.mark.parametrize("depth", list(DEPTHS))
@pytest.mark.parametrize("length", [1, 2, 512, 513, 2047, 2048, 2049, 8192, 8193, 20_011, 65_536, 65_537])
def test_one_long_list(gpu_lib, length, depth):
    """One tile holds `length` entries, its neighbours a few or none."""
    R = H.raster()
    g = gs_inputs.rng(length + len(depth))
    cams = [_Cam(75, 41)]  # 5 x 3 tiles
    n = length + 40
    boxes = np.zeros((n, 4), dtype=np.int64)
    boxes[:] = (16, 31, 16, 31)
    boxes[length:] = (1, 0, 1, 0)  # not drawn
    boxes[length:length + 7] = (32, 74, 0, 40)
    p = g.permutation(n)
    z = DEPTHS[depth](g, n)
    st = _compare(R, _projected(R, cams, boxes[p], z), cams, n, f"list of {length}, {depth}")
    assert st.max_list >= length
    assert st.list_slices == (0 if length <= 2048 else 1 if length <= 8192 else -(-length // 4096))


@pytest.mark.parametrize("n,sizes", [(1, [(16, 16)]), (300, [(17, 16)]), (257, [(2100, 1100), (33, 700)]),
                                     (5000, [(640, 480), (64, 48), (801, 603)]), (300_001, [(320, 200)])])
def test_mixed_boxes_and_views(gpu_lib, n, sizes):
    """Random boxes from one pixel to the whole image, several views, more tiles
    than one table holds (2100 x 1100: 9,108 tiles), some records not drawn."""
    R = H.raster()
    g = gs_inputs.rng(n)
    cams = [_Cam(w, h) for w, h in sizes]
    boxes = []
    for w, h in sizes:
        c = np.stack([g.integers(0, w, n), g.integers(0, h, n)], 1)
        half = np.where(g.uniform(size=n) < 0.01, 4096, g.integers(0, 24, n))
        b = np.stack([np.maximum(c[:, 0] - half, 0), np.minimum(c[:, 0] + half, w - 1),
                      np.maximum(c[:, 1] - half, 0), np.minimum(c[:, 1] + half, h - 1)], 1)
        if n > 100_000:
            b[:, :] = np.stack([c[:, 0], c[:, 0], c[:, 1], c[:, 1]], 1)
        b[g.uniform(size=n) < 0.2] = (1, 0, 1, 0)
        boxes.append(b)
    z = np.concatenate([DEPTHS["spread"](g, n) for _ in sizes])
    _compare(R, _projected(R, cams, np.concatenate(boxes), z), cams, n, f"mixed n={n} {sizes}")


def test_records_in_no_order(gpu_lib):
    """Small boxes at random places of a large view: the pairs are not counted
    by tile, and the lists come from the radix sort; sorted by place they are."""
    R = H.raster()
    g = gs_inputs.rng(12)
    cams = [_Cam(1920, 1080)]
    n = 40_000
    x, y = g.integers(0, 1900, n), g.integers(0, 1060, n)
    z = DEPTHS["spread"](g, n)
    boxes = np.stack([x, x + 12, y, y + 12], 1)
    assert _compare(R, _projected(R, cams, boxes, z), cams, n, "no order").max_list == 0
    o = np.lexsort((x // 120, y // 120))
    assert _compare(R, _projected(R, cams, boxes[o], z[o]), cams, n, "by place").max_list > 0


def test_culled_scene_and_views(gpu_lib):
    """A projected scene in two views, with and without culled tiles, into
    reused buffers that hold an earlier call's lists."""
    R = H.raster()
    wl = gs_inputs.small_cube(seed=4, n=6000, width=203, height=131)
    cams = [wl.cameras[0], gs_inputs.look_at((1.0, 0.5, 3.0), (0, 0, 0), 97, 260)]
    ds = R.DeviceScene.from_numpy(wl.scene)
    bufs = R.StepBuffers()
    for cull in (False, True, False):
        proj = R.project(ds, cams, R.RasterOpts(tile_cull=cull))
        _compare(R, proj, cams, ds.n, f"cull={cull}")
        offsets, st = R.bin_count(proj, cams, ds.n)
        ref = R.bin_sort(proj, cams, ds.n, offsets, st)
        for _ in range(2):
            got = R.bin_step(proj, cams, ds.n, bufs)
            torch.cuda.synchronize()
            for f in ("vals", "ranges", "order", "offsets"):
                assert torch.equal(getattr(got, f), getattr(ref, f)), f


def test_look_back_sort_stays_selectable(gpu_lib):
    """With the look-back sort selected the lists come from it (and its error
    flag), and are the same."""
    from paper_2411_12788_amd import _lib as L
    R = H.raster()
    wl = gs_inputs.small_cube(seed=6, n=3000)
    ds = R.DeviceScene.from_numpy(wl.scene)
    proj = R.project(ds, wl.cameras, R.RasterOpts())
    a = R.bin(proj, wl.cameras, ds.n)
    L.lib().gs_sort_set_algorithm(L.GS_SORT_LOOKBACK)
    try:
        b = R.bin(proj, wl.cameras, ds.n)
    finally:
        L.lib().gs_sort_set_algorithm(L.GS_SORT_PRESCAN)
    torch.cuda.synchronize()
    assert a.stats.max_list > 0 and b.stats.max_list == 0
    for f in ("vals", "ranges", "order", "offsets"):
        assert torch.equal(getattr(a, f), getattr(b, f)), f


def test_argument_errors(gpu_lib):
    from paper_2411_12788_amd import _lib as L
    R = H.raster()
    lib = L.lib()
    cams = R.cameras([gs_inputs.look_at((0, 0, 4), (0, 0, 0), 16, 16)])
    fake = ctypes.c_void_p(0x1000)
    st = L.BinStats()
    st.n_isect, st.tiles_total, st.max_list = 10, 1, 10
    proj = L.Projected(fake, fake, 0.0)
    cb, sb = lib.gs_bin_count_workspace_size(10), lib.gs_bin_sort_workspace_size(10)

    def lists(proj=ctypes.byref(proj), vals=fake, ranges=fake, cws=fake, cb=cb, sb=sb, stats=st):
        return lib.gs_bin_lists(proj, cams, 1, 10, fake, ctypes.byref(stats), None, vals, ranges, fake, cws, cb, fake,
                                sb, None)
    assert lists(proj=None) == L.GS_ERR_NULL and lists(vals=None) == L.GS_ERR_NULL
    assert lists(ranges=None) == L.GS_ERR_NULL and lists(cws=None) == L.GS_ERR_NULL
    assert lists(cb=cb - 1) == L.GS_ERR_CAPACITY and lists(sb=sb - 1) == L.GS_ERR_CAPACITY
    other = L.BinStats()
    other.n_isect, other.tiles_total, other.max_list = 10, 2, 10
    assert lists(stats=other) == L.GS_ERR_SHAPE
    assert lib.gs_bin_tiles(ctypes.byref(proj), cams, 1, 10, fake, ctypes.byref(st), fake, fake, fake, cb - 1,
                            None) == L.GS_ERR_CAPACITY
