"""What raster.bin reads back after the lists are made: the status flag of the
look-back sort (raised when a wait gives up), nothing with the default sort,
and the same lists either way; cameras given as objects or as the library's
array; and the render's gradients when colour's gradient is the only one or
comes with none at all."""
import pytest
import torch

import gs_inputs
from tests import gpu_helpers as H

pytestmark = pytest.mark.gpu


def _scene(n=3000):
    wl = gs_inputs.small_cube(seed=3, n=n, width=112, height=96)
    return wl, H.raster().DeviceScene.from_numpy(wl.scene)


@pytest.mark.parametrize("algorithm", [0, 1])
@pytest.mark.parametrize("own_stream", [False, True])
def test_bin_lists_do_not_depend_on_the_check(gpu_lib, algorithm, own_stream):
    from paper_2411_12788_amd import _lib as L
    R = H.raster()
    wl, ds = _scene()
    stream = torch.cuda.Stream() if own_stream else None
    if stream is not None:
        stream.wait_stream(torch.cuda.current_stream())
    assert L.lib().gs_sort_set_algorithm(algorithm) == L.GS_OK
    try:
        assert L.lib().gs_sort_waits() == algorithm
        proj = R.project(ds, wl.cameras, R.RasterOpts(), stream=stream)
        got = R.bin(proj, wl.cameras, ds.n, stream=stream)
        as_array = R.bin(proj, R.cameras(wl.cameras), ds.n, stream=stream)
    finally:
        L.lib().gs_sort_set_algorithm(0)
    torch.cuda.synchronize()
    ref = R.bin(R.project(ds, wl.cameras, R.RasterOpts()), wl.cameras, ds.n)
    torch.cuda.synchronize()
    for b in (got, as_array):
        assert torch.equal(b.vals, ref.vals) and torch.equal(b.ranges, ref.ranges) and torch.equal(b.order, ref.order)


def test_gradients_of_colour_alone_and_of_none(gpu_lib):
    from paper_2411_12788_amd import autograd as A
    wl, ds = _scene()
    leaves = [t.clone().requires_grad_() for t in (ds.means, ds.scales, ds.quats, ds.opacity, ds.sh)]
    color, depth, imax = A.rasterize(*leaves, wl.cameras, deterministic=True)
    assert not depth.requires_grad and not imax.requires_grad
    dl = torch.randn_like(color)
    one = torch.autograd.grad(color, leaves, dl, retain_graph=True)
    # the same through a graph that also reaches the outputs without gradient
    two = torch.autograd.grad((color * dl).sum() + 0.0 * depth.sum(), leaves)
    for a, b in zip(one, two):
        assert torch.equal(a, b)
    # a backward that passes no gradient gives zeros
    ctx_grads = A.RasterizeFn.apply(*leaves, list(wl.cameras), H.raster().RasterOpts(), 3, None, False, None, True)
    got = ctx_grads[0].grad_fn.apply(None, None, None)
    for g in got[:5]:
        assert not g.any()
