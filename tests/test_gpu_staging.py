"""Staging slots that hold no list entry.  The compositing kernels stage 192 or
256 entries at a time, and the groups of a wave walk to the longest of their
streams, so a group reads past the end of its own, in the last round also slots
beyond the list.  Nothing in such a slot may reach a result: here the record
buffer is full of NaN before the projection, which leaves the rows of records
that are not drawn as they are, row 0 among them.  Every output is finite and
equals the oracle's."""
import numpy as np
import pytest
import torch

import gs_inputs
import oracle
from tests import gpu_helpers as H
from tests.oracle_scenes import identity_camera, scene_from

pytestmark = pytest.mark.gpu

SIDE, F0 = 48, 60.0  # nine tiles


def _np(t):
    return t.detach().cpu().numpy()


def _scene(n, seed, others):
    """n small Gaussians inside the middle tile, five in six of them around one
    corner, so that its 4x4 groups have streams of very different lengths;
    `others`: one more in each of the other tiles.  Gaussian 0 is behind the
    camera."""
    g = gs_inputs.rng(seed)
    uv = g.uniform(20.0, 28.0, size=(n, 2))
    corner = g.uniform(size=n) < 5 / 6
    uv[corner] = 20.0 + 2.0 * g.uniform(size=(corner.sum(), 2))
    z = g.uniform(2.0, 6.0, size=n)
    r = g.uniform(0.2, 0.7, size=(n, 3))  # pixels
    opacity = g.uniform(0.01, 0.03, size=n)
    if others:
        c = np.array([(8.0 + 16 * x, 8.0 + 16 * y) for x in range(3) for y in range(3) if (x, y) != (1, 1)])
        uv, z = np.concatenate([uv, c]), np.concatenate([z, np.full(8, 3.0)])
        r, opacity = np.concatenate([r, np.full((8, 3), 0.5)]), np.concatenate([opacity, np.full(8, 0.5)])
    means = np.stack([(uv[:, 0] - SIDE / 2) / F0 * z, (uv[:, 1] - SIDE / 2) / F0 * z, z], 1)
    means = np.concatenate([[[0.0, 0.0, -1.0]], means])
    m = len(means)
    scales = np.concatenate([[[0.1] * 3], r * z[:, None] / F0])
    sh = gs_inputs.rng(seed + 1).normal(0.0, 0.2, size=(16, 3, m)).astype(np.float32)
    return scene_from(means, scales, g.normal(size=(m, 4)), np.concatenate([[0.5], opacity]), sh=sh, degree=3)


@pytest.mark.parametrize("form,n", [(f, n) for f in ("whole", "rows") for n in (257, 300, 449, 600)] +
                         [("group", 2100), ("group", 2305)])
def test_slots_without_an_entry(gpu_lib, form, n):
    """whole: no tile order.  rows: the one tile with entries, split with four
    entries side by side.  group: one long list among tiles with entries, the
    forward's split work item with its group in lanes 0-15."""
    R = H.raster()
    sc = _scene(n, n, others=form == "group")
    cam = identity_camera(SIDE, SIDE, F0)
    ds = R.DeviceScene.from_numpy(sc)
    Pn = SIDE * SIDE
    p = oracle.Params.of(sc)
    dldc = gs_inputs.normal_image(3, Pn, 61, scale=1.0 / Pn)
    mask = gs_inputs.bernoulli_mask(sc.n, 0.25, 62)
    for depth_mode in (0, 1, 2):
        opts, o = R.RasterOpts(depth_mode=depth_mode), oracle.Opts(depth_mode=depth_mode)
        buffers = R.StepBuffers()
        buffers.take("rec", sc.n, torch.float32, "cuda", (16,)).fill_(float("nan"))
        buffers.store["rec"].fill_(float("nan"))
        proj = R.project(ds, [cam], opts, buffers=buffers)
        assert torch.isnan(proj.rec[0]).all()  # row 0 is not drawn, and not written
        binned = R.bin(proj, [cam], sc.n)
        rng = _np(binned.ranges).reshape(-1, 2)
        assert (rng[:, 1] - rng[:, 0]).max() == n and ((rng[:, 1] - rng[:, 0]) > 0).sum() == (9 if form == "group" else 1)
        if form == "whole":
            binned.order = None
        orc = oracle.forward_view(p, cam, o)
        for accumulate in (False, True):
            print(f"{form}, list of {n}, depth mode {depth_mode}, accumulate {accumulate}", flush=True)
            acc = R.alloc_accum(sc.n) if accumulate else None
            frame = R.render_forward(ds, proj, binned, [cam], opts, accum=acc)
            for k in ("color", "depth", "t_final"):
                assert torch.isfinite(getattr(frame, k)).all(), (k, depth_mode, accumulate)
            flips, _ = H.compare_forward(frame, orc, slice(0, Pn), f"{form} {n}", p, cam, o)
            if accumulate:
                H.check_accum(acc, p, cam, orc["proj"], orc["order"], o, flips, sc.n, f"{form} {n}")
        if depth_mode:
            continue
        for m in (None, mask):
            og, _ = H.backward_views(p, [cam], o, [dldc.T.astype(np.float64)], active=m, flips=[flips])
            for det in (False, True):
                grads, g2d = R.render_backward(ds, proj, binned, [cam], opts, frame, torch.from_numpy(dldc).cuda(),
                                               None if m is None else torch.from_numpy(m).cuda(), deterministic=det)
                assert torch.isfinite(g2d).all(), (m is None, det)
                for k in og:
                    got = _np(grads[k])[..., :sc.n]
                    assert np.isfinite(got).all() and H.rel_l2(got, og[k]) <= H.GRAD_REL_L2, (k, m is None, det)


def test_flushed_rounds_leave_no_offsets(gpu_lib):
    """Three rounds of 192 entries in one tile.  What the workgroup leaves in LDS
    between two of them must not be taken for an offset: in the first round
    walked (the list's last) entry 32 has a record index whose low byte, 216, is
    no staging slot, and lands where the stream of group 1 of the first wave
    begins; that group has no entry in the second round, in which the bytes that
    a slot 216 would be read from are not a number; its one entry is in the
    third."""
    R = H.raster()
    n, side, f = 1024, 16, 40.0
    cam = identity_camera(side, side, f)
    at = np.zeros((576, 2), dtype=int)
    at[:] = (3, 2)                        # quarter and group of each list position
    for k in (10, 20, 30, 127):
        at[384 + k] = (0, 2)
    for k in (1, 2, 130):
        at[192 + k] = (0, 2)
    at[50] = (0, 1)
    index = np.arange(576)
    index[384 + 32] = 2 * 256 + 216       # 728: beyond the others
    q, grp = at[:, 0], at[:, 1]
    u, v = 8 * (q & 1) + 4 * (grp & 1) + 2.0, 8 * (q >> 1) + 4 * (grp >> 1) + 2.0
    z = 2.0 + 0.01 * np.arange(576)
    g = gs_inputs.rng(9)
    means, scales, opacity = np.tile((0.0, 0.0, 3.0), (n, 1)), np.full((n, 3), 0.01), np.zeros(n)
    means[index] = np.stack([(u - side / 2) / f * z, (v - side / 2) / f * z, z], 1)
    scales[index] = g.uniform(0.1, 0.3, size=(576, 3)) * z[:, None] / f
    opacity[index] = np.where((at == (3, 2)).all(1), g.uniform(0.012, 0.016, size=576), 0.05)
    opacity[index[50]] = 0.3
    sh = gs_inputs.rng(10).normal(0.0, 0.2, size=(16, 3, n)).astype(np.float32)
    sc = scene_from(means, scales, g.normal(size=(n, 4)), opacity, sh=sh, degree=3)
    ds = R.DeviceScene.from_numpy(sc)
    opts, o, Pn = R.RasterOpts(), oracle.Opts(), side * side
    proj = R.project(ds, [cam], opts)
    binned = R.bin(proj, [cam], n)
    assert np.array_equal(_np(binned.vals), index)
    frame = R.render_forward(ds, proj, binned, [cam], opts)
    assert int(frame.last.max()) == 576  # the rounds begin at the list's end
    p = oracle.Params.of(sc)
    orc = oracle.forward_view(p, cam, o)
    flips, _ = H.compare_forward(frame, orc, slice(0, Pn), "flushed rounds", p, cam, o)
    dldc = gs_inputs.normal_image(3, Pn, 63, scale=1.0 / Pn)
    og, _ = H.backward_views(p, [cam], o, [dldc.T.astype(np.float64)], flips=[flips])
    for mask in (None, np.ones(n, dtype=np.uint8)):
        grads, g2d = R.render_backward(ds, proj, binned, [cam], opts, frame, torch.from_numpy(dldc).cuda(),
                                       None if mask is None else torch.from_numpy(mask).cuda())
        assert torch.isfinite(g2d).all()
        for k in og:
            assert H.rel_l2(_np(grads[k])[..., :n], og[k]) <= H.GRAD_REL_L2, k
