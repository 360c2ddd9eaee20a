"""Records whose own tile counts (bin.w, which size the lists) are not what a
walk over their boxes gives: projected with tile culling and binned without,
or changed by hand.  The binning then takes the radix sort, which keeps every
record inside its own slots; lists and ranges stay inside the pairs counted and
nothing is written past them."""
import ctypes

import numpy as np
import pytest
import torch

import gs_inputs
from paper_2411_12788_amd import _lib as L
from tests import gpu_helpers as H

pytestmark = pytest.mark.gpu

GUARD, MARK = 65536, 0x5A5A5A5A


def _scene():
    wl = gs_inputs.uniform_cube_scene(4096, 3)
    return wl, [gs_inputs.look_at((0, 0, 4), (0, 0, 0), 128, 128), gs_inputs.look_at((3, 1, 2.5), (0, 0, 0), 100, 70)]


def _gs_bin(R, proj, cams, n):
    """gs_bin into buffers of exactly the pairs that the records count, with
    GUARD marked words after vals, keys and ranges."""
    lib, V, dev = L.lib(), len(cams), "cuda"
    pairs = int(proj.bin[: V * n, 3].clamp(min=0).sum())
    tiles = R.tiles_total(cams)
    marked = lambda words: torch.full((words + GUARD,), MARK, dtype=torch.int32, device=dev)
    vals, keys, ranges, order = marked(pairs), marked(2 * pairs), marked(2 * tiles), marked(tiles)
    offsets = torch.empty(V * n, dtype=torch.int32, device=dev)
    cws = torch.zeros(lib.gs_bin_count_workspace_size(V * n), dtype=torch.uint8, device=dev)
    sws = torch.zeros(lib.gs_bin_sort_workspace_size(pairs), dtype=torch.uint8, device=dev)
    st, pc = L.BinStats(), proj.c()
    p = lambda t: ctypes.c_void_p(t.data_ptr())
    rc = lib.gs_bin(ctypes.byref(pc), R.cameras(cams), V, n, p(offsets), ctypes.byref(st), p(keys), p(vals), pairs,
                    p(ranges), p(order), p(cws), cws.numel(), p(sws), sws.numel(), R._stream())
    torch.cuda.synchronize()
    assert rc == L.GS_OK and st.n_isect == pairs
    for name, t, words in (("vals", vals, pairs), ("keys", keys, 2 * pairs), ("ranges", ranges, 2 * tiles),
                           ("order", order, tiles)):
        assert bool((t[words:] == MARK).all()), f"{name} written past its end"
    r = ranges[: 2 * tiles].cpu().numpy().view(np.uint32).reshape(-1, 2)
    assert (r[:, 0] <= r[:, 1]).all() and r.max(initial=0) <= pairs
    return st, r


@pytest.mark.parametrize("case", ["consistent", "culled, binned without", "fewer", "more"])
def test_counts_that_differ_from_the_walk(gpu_lib, case):
    R = H.raster()
    sc, cams = _scene()
    ds = R.DeviceScene.from_numpy(sc).in_spatial_order()[0]
    proj = R.project(ds, cams, R.RasterOpts(tile_cull=case == "culled, binned without"))
    w = proj.bin[:, 3]
    some = w > 1
    some[torch.arange(w.numel(), device=w.device) % 7 != 0] = False
    assert int(some.sum()) > 20
    if case == "fewer":
        w[some] -= 1
    elif case == "more":
        w[some] += 1
    elif case != "consistent":
        proj.tile_cull_log2_alpha = 0.0
    print(case, flush=True)
    st, r = _gs_bin(R, proj, cams, sc.n)
    if case == "consistent":
        assert st.max_list > 0 and (r[:, 1] - r[:, 0]).sum() == st.n_isect
    else:
        assert st.max_list == 0 and st.list_slices == 0
