"""The rasterizer's own workloads as timed cases: training steps, forward-only
renders as the server runs them, and the once-in-a-while work on the set of
Gaussians, each through the package's public entry points.

A case is a dict of plain values; `prepare` makes what a user's program holds
before the call (scene, cameras, targets, reused buffers), `run` makes one
pass, `exact` gives the same outputs from plain float64 torch where that is
affordable.

Kinds
  step      one differentiable render through autograd.rasterize and its
            gradients: what a training script with its own optimizer calls
  loop      one step of a training loop that keeps its buffers: clears,
            projection, binning, forward with the per-Gaussian accumulations,
            loss gradient, masked backward
  render    forward-only views with the server's options and reused buffers
  criteria  visibility, critical set, blur split and simplification sampling
            from accumulated importances
  densify   density control: selection, clone, split, then the reorder that
            follows a change of the set

Scenes are Gaussians on twenty random spheres and plane patches ("surfaces",
`half` is the half-width of the region, seen from three times as far), or in
a cube, with the scale, opacity and colour distributions of the repository's
synthetic inputs.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2411_12788_amd import autograd, densify, raster

RESOLUTIONS = [(640, 480), (800, 600), (1024, 768), (1280, 720),
               (1280, 960), (1440, 1080), (1600, 900), (1600, 1200)]
EXACT_PAIRS = 80_000_000  # Gaussians x pixels up to which exact() composites every pair
THRESHOLD, SCALE_THRESHOLD = 2e-4, 0.01  # density control


def listed():
    return [
        # the smallest call: a unit-test sized scene, where launches, the pair
        # count's round trip and host work are what a user waits for
        dict(name="step_4k_128", kind="step", scene="cube", gaussians=4096, views=1, width=128, height=128, half=1.0,
             degree=3, active=0.0, save_lists=False, deterministic=False),
        # one training view of an early set at a usual photo size
        dict(name="step_500k_1245x825", kind="step", scene="surfaces", gaussians=500_000, views=1, width=1245,
             height=825, half=2.0, degree=3, active=0.0, save_lists=False, deterministic=False),
        # reproducible training: ordered reduction, lists kept, odd sizes
        dict(name="step_300k_ordered", kind="step", scene="surfaces", gaussians=300_001, views=1, width=801, height=603,
             half=2.0, degree=3, active=0.25, save_lists=True, deterministic=True),
        # the batched differentiable render: sixteen views of mixed size at once
        dict(name="step_1m_16views", kind="step", scene="surfaces", gaussians=1_000_000, views=16, width=0, height=0,
             half=2.0, degree=3, active=0.0, save_lists=False, deterministic=False),
        # the dense phase of training: a large set over a wide region, a
        # quarter of it active, accumulations on
        dict(name="loop_3m_1080p", kind="loop", scene="surfaces", gaussians=3_000_000, views=1, width=1920, height=1080,
             half=10.0, degree=3, active=0.25),
        # warm-up phase of training: low SH degree, everything active, a small odd image
        dict(name="loop_100k_637x479", kind="loop", scene="surfaces", gaussians=100_003, views=1, width=637, height=479,
             half=2.0, degree=1, active=0.0),
        # served views: a light scene, a heavy one, a batch of views of one scene
        dict(name="render_200k_800", kind="render", scene="surfaces", gaussians=200_000, views=1, width=800, height=800,
             half=2.0, degree=3),
        dict(name="render_3m_1080p", kind="render", scene="surfaces", gaussians=3_000_000, views=1, width=1920,
             height=1080, half=2.0, degree=3),
        dict(name="render_1500k_4views", kind="render", scene="surfaces", gaussians=1_500_000, views=4, width=1280,
             height=720, half=2.0, degree=3),
        # culling and simplification criteria over a few views' importances
        dict(name="criteria_1m_4views", kind="criteria", gaussians=1_000_000, views=4),
        # density control and the reorder after it
        dict(name="densify_1m", kind="densify", scene="surfaces", gaussians=1_000_000, half=2.0, selected=0.08),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step"] * 3 + ["loop"] * 3 + ["render"] * 3 + ["criteria", "densify"])
    if kind == "criteria":
        return dict(kind=kind, gaussians=_log_uniform(rng, 20_000, 2_000_000), views=rng.randint(1, 8))
    if kind == "densify":
        return dict(kind=kind, scene="surfaces", gaussians=_log_uniform(rng, 20_000, 1_500_000), half=2.0,
                    selected=round(rng.uniform(0.01, 0.2), 3))
    small = rng.random() < 0.25
    if small:
        n, w, h = _log_uniform(rng, 300, 8000), rng.randint(17, 100), rng.randint(16, 100)
        case = dict(kind=kind, scene="cube", gaussians=n, views=rng.randint(1, 2), width=w, height=h, half=1.0)
    else:
        n = _log_uniform(rng, 50_000, 3_000_000 if kind != "step" else 1_000_000)
        w, h = _log_uniform(rng, 200, 1920), _log_uniform(rng, 150, 1080)
        views = rng.choice([1, 1, 1, 2, 3, 5]) if n <= 1_000_000 else 1
        case = dict(kind=kind, scene="surfaces", gaussians=n, views=views, width=w, height=h,
                    half=rng.choice([2.0, 2.0, 5.0, 10.0]))
    case["degree"] = rng.choice([3, 3, 3, 0, 1, 2])
    if kind != "render":
        case["active"] = rng.choice([0.0, 0.25, 0.6])
    if kind == "step":
        case["save_lists"] = rng.random() < 0.5
        case["deterministic"] = rng.random() < 0.2
    return case


# --------------------------------------------------------------------------
# inputs
# --------------------------------------------------------------------------
class Camera:
    """Pinhole camera looking at the origin (x right, y down, z forward)."""

    def __init__(self, eye, width, height, fov_x_deg=60.0):
        eye = np.asarray(eye, dtype=np.float64)
        zc = -eye / np.linalg.norm(eye)
        up = np.array([0.0, 1.0, 0.0]) if abs(zc[1]) < 0.999 else np.array([0.0, 0.0, 1.0])
        xc = np.cross(zc, up)
        xc /= np.linalg.norm(xc)
        self.R = np.stack([xc, np.cross(zc, xc), zc]).astype(np.float32)
        self.t = (-(self.R.astype(np.float64) @ eye)).astype(np.float32)
        self.width, self.height = int(width), int(height)
        self.fx = self.fy = float(np.float32(width / 2.0 / math.tan(math.radians(fov_x_deg) / 2.0)))
        self.cx, self.cy = width / 2.0, height / 2.0


def _cameras(case, seed):
    g = np.random.default_rng(seed + 1)
    out = []
    for k in range(case["views"]):
        d = g.normal(size=3)
        d /= np.linalg.norm(d)
        w, h = (case["width"], case["height"]) if case["width"] else RESOLUTIONS[(k // 2) % len(RESOLUTIONS)]
        out.append(Camera((4.0 if case["scene"] == "cube" else 3.0 * case["half"]) * d, w, h))
    return out


def _scene(case, seed):
    """(means, scales, quats, opacity, sh) float32 planes on the GPU."""
    n = case["gaussians"]
    g = torch.Generator(device="cuda").manual_seed(seed)

    def normal(*shape):
        return torch.randn(shape, device="cuda", generator=g)

    if case["scene"] == "cube":
        means = (torch.rand((3, n), device="cuda", generator=g) * 2 - 1) * case["half"]
        scales = torch.exp(normal(3, n) * 0.5 - 3.5)
    else:
        h = np.random.default_rng(seed)
        sphere = h.uniform(size=20) < 0.5
        centre = h.uniform(-case["half"], case["half"], size=(20, 3))
        radius = h.uniform(0.5, 3.0, size=20)
        e1, e2 = np.zeros((20, 3)), np.zeros((20, 3))
        for s in range(20):
            q, _ = np.linalg.qr(h.normal(size=(3, 3)))
            e1[s], e2[s] = q[:, 0], q[:, 1]

        def dev(a):
            return torch.from_numpy(np.ascontiguousarray(a, dtype=np.float32)).cuda()

        which = torch.arange(n, device="cuda") * 20 // n
        d = normal(3, n)
        ab = torch.rand((2, n), device="cuda", generator=g) * 2 - 1
        flat = dev(e1).T[:, which] * ab[0] + dev(e2).T[:, which] * ab[1]
        unit = torch.where(dev(sphere)[which] > 0.5, d / d.norm(dim=0, keepdim=True), flat)
        means = dev(centre).T[:, which] + dev(radius)[which] * unit + 0.02 * normal(3, n)
        scales = torch.exp(normal(3, n) * 0.7 - 5.0)
    quats = normal(4, n)
    quats = quats / quats.norm(dim=0, keepdim=True)
    opacity = torch.sigmoid(normal(n))
    sh = 0.05 * normal(16, 3, n)
    sh[0] = 0.5 + 0.2 * normal(3, n)
    return [t.contiguous() for t in (means, scales, quats, opacity, sh)]


def _device_scene(case, seed):
    """The scene as a program keeps it: in the library's spatial order."""
    s = raster.DeviceScene(*_scene(case, seed), case.get("degree", 3))
    return s.in_spatial_order()[0]


def _mask(case, seed):
    if not case["active"]:
        return None
    g = torch.Generator(device="cuda").manual_seed(seed + 2)
    return (torch.rand(case["gaussians"], device="cuda", generator=g) < case["active"]).to(torch.uint8)


def _importance_like(views, n, g):
    v = torch.exp(2.0 * torch.randn((views, n), device="cuda", generator=g))
    return torch.where(torch.rand((views, n), device="cuda", generator=g) < 0.4, torch.zeros_like(v), v)


def prepare(case, seed):
    kind = case["kind"]
    g = torch.Generator(device="cuda").manual_seed(seed + 3)
    n = case["gaussians"]
    if kind == "criteria":
        wmax = 0.99 * torch.rand(n, device="cuda", generator=g) ** 2
        area = torch.where(torch.rand(n, device="cuda", generator=g) < 0.5, 0.0,
                           20.0 * torch.rand(n, device="cuda", generator=g) ** 3 + 1).to(torch.int32)
        expo = -torch.log1p(-torch.rand(n, device="cuda", generator=g))
        return dict(case=case, importance=_importance_like(case["views"], n, g), wmax=wmax, area=area, expo=expo)
    if kind == "densify":
        scene = _device_scene(dict(case, degree=3), seed)
        count = torch.randint(1, 17, (n,), device="cuda", generator=g, dtype=torch.int32)
        # mean gradient norms: the given share above the threshold, a third of
        # them Gaussians large enough to be split
        mean = THRESHOLD * torch.rand(n, device="cuda", generator=g)
        big = scene.scales.max(0)[0] > SCALE_THRESHOLD
        hot = int(n * case["selected"])
        for rows, k in ((big.nonzero()[:, 0], hot // 3), ((~big).nonzero()[:, 0], hot - hot // 3)):
            rows = rows[torch.randperm(rows.numel(), device="cuda", generator=g)[:k]]
            mean[rows] = THRESHOLD * (2 + torch.rand(k, device="cuda", generator=g))
        normals = torch.randn((2, 3, 2 * n), device="cuda", generator=g)
        return dict(case=case, scene=scene, count=count, norm=count * mean, normals=normals)
    scene = _device_scene(case, seed)
    cams = _cameras(case, seed)
    P = sum(c.width * c.height for c in cams)
    st = dict(case=case, scene=scene, cams=cams)
    if kind == "render":
        st["opts"] = raster.RasterOpts(tile_cull=True)
        st["buffers"] = raster.StepBuffers()
        return st
    st["active"] = _mask(case, seed)
    if kind == "step":
        st["leaves"] = [t.requires_grad_() for t in (scene.means, scene.scales, scene.quats, scene.opacity, scene.sh)]
        st["dl"] = torch.randn((3, P), device="cuda", generator=g) / P
    else:
        st["target"] = torch.rand((3, P), device="cuda", generator=g)
        st["opts"] = raster.RasterOpts()
        st["buffers"] = raster.StepBuffers()
        st["acc"] = raster.alloc_accum(n)
        st["loss"] = torch.zeros(1, device="cuda")
        st["dl"] = torch.empty((3, P), device="cuda")
        st["grads"] = raster.alloc_grads(n)
        st["grad2d"] = torch.empty((len(cams) * n, 9), device="cuda")
        st["frame"] = None
    return st


# --------------------------------------------------------------------------
# one pass
# --------------------------------------------------------------------------
GRADS = ("means", "scales", "quats", "opacity", "sh")


def run(s):
    case = s["case"]
    return dict(step=_run_step, loop=_run_loop, render=_run_render, criteria=_run_criteria,
                densify=_run_densify)[case["kind"]](case, s)


def _run_step(case, s):
    color, depth, imax = autograd.rasterize(*s["leaves"], s["cams"], sh_degree=case["degree"], active=s["active"],
                                            save_lists=case["save_lists"], deterministic=case["deterministic"])
    grads = torch.autograd.grad(color, s["leaves"], s["dl"])
    return dict(color=color.detach(), depth=depth, imax=imax, **{"d_" + k: v for k, v in zip(GRADS, grads)})


def _run_loop(case, s):
    scene, cams, opts, acc = s["scene"], s["cams"], s["opts"], s["acc"]
    for t in (acc["importance"], acc["wmax"], acc["area"], s["loss"]):
        raster.fill_u32(t, 0)
    proj = raster.project(scene, cams, opts, buffers=s["buffers"])
    binned = raster.bin_step(proj, cams, scene.n, s["buffers"])
    s["frame"] = f = raster.render_forward(scene, proj, binned, cams, opts, accum=acc, out=s["frame"])
    raster.l1_loss_grad(f.color, s["target"], s["dl"], s["loss"])
    raster.render_backward(scene, proj, binned, cams, opts, f, s["dl"], s["active"], s["grads"], s["grad2d"])
    return dict(color=f.color, depth=f.depth, imax=f.imax, t_final=f.t_final, last=f.last, n_contrib=f.n_contrib,
                hit=f.hit, loss=s["loss"], **acc, **{"d_" + k: s["grads"][k] for k in GRADS})


def _run_render(case, s):
    scene, cams, opts = s["scene"], s["cams"], s["opts"]
    proj = raster.project(scene, cams, opts, buffers=s["buffers"])
    binned = raster.bin_step(proj, cams, scene.n, s["buffers"])
    f = raster.render_forward(scene, proj, binned, cams, opts, extras=False)
    return dict(color=f.color, depth=f.depth, imax=f.imax, t_final=f.t_final)


def _run_criteria(case, s):
    visible, tau = densify.visibility(s["importance"])
    critical, ctau = densify.critical(s["area"], s["wmax"])
    blur = densify.blur_split(s["area"], 300, 400)
    keep, count = densify.sample(s["importance"][0], s["expo"], case["gaussians"] // 3, s["area"])
    return dict(visible=visible, tau=tau, critical=critical, critical_tau=ctau, blur=blur, keep=keep, count=count)


def _run_densify(case, s):
    scene = s["scene"]
    clone, split = densify.densify_select(s["norm"], s["count"], scene.scales, THRESHOLD, SCALE_THRESHOLD)
    grown, cloned = densify.clone(scene, clone)
    select = torch.nn.functional.pad(split, (0, grown.n - scene.n))
    normals = s["normals"][:, :, :grown.n].contiguous()
    out, halved = densify.split(grown, select, normals)
    out, _, perm = densify.reorder(out)
    return dict(means=out.means, scales=out.scales, quats=out.quats, opacity=out.opacity, sh=out.sh, perm=perm,
                cloned=cloned, halved=halved)


# --------------------------------------------------------------------------
# what a pass cannot do without
# --------------------------------------------------------------------------
def work(case):
    """Each input read once, each output written once.  Operations: the
    projection's and the per-pixel compositing's (about twenty Gaussians a
    pixel), their backward twice that."""
    n = case["gaussians"]
    if case["kind"] == "criteria":
        return dict(bytes=n * (case["views"] * 5 + 4 + 4 + 4 + 3), flops=4.0 * n * (case["views"] + 2))
    if case["kind"] == "densify":
        m = int(n * (1 + 2 * case["selected"]))
        return dict(bytes=236 * (n + m) + 12 * n + 4 * m, flops=40.0 * m)
    V = case["views"]
    if case["width"]:
        P = V * case["width"] * case["height"]
    else:
        P = sum(w * h for w, h in (RESOLUTIONS[(k // 2) % len(RESOLUTIONS)] for k in range(V)))
    K = (case["degree"] + 1) ** 2
    params = 4 * (11 + 3 * K)
    fwd = 600.0 * V * n + 20 * 30.0 * P
    if case["kind"] == "render":
        return dict(bytes=n * params + 28 * P, flops=fwd)
    if case["kind"] == "step":
        return dict(bytes=n * (params + 236) + P * (12 + 8 + 12), flops=3 * fwd)
    return dict(bytes=n * (params + 236 + 12) + P * (33 + 24), flops=3 * fwd)


# --------------------------------------------------------------------------
# float64 reference
# --------------------------------------------------------------------------
C0, C1 = 0.28209479177387814, 0.4886025119029199


def _sh_basis(d, degree):
    x, y, z = d
    one = torch.ones_like(x)
    b = [C0 * one]
    if degree >= 1:
        b += [C1 * y, C1 * z, C1 * x]
    if degree >= 2:
        a, c, e = 1.0925484305920792, 0.31539156525252005, 0.5462742152960396
        b += [a * x * y, a * y * z, c * (2 * z * z - x * x - y * y), a * x * z, e * (x * x - y * y)]
    if degree >= 3:
        a, c, e, f, g = (0.5900435899266435, 2.890611442640554, 0.4570457994644658, 0.3731763325901154,
                         1.445305721320277)
        b += [a * y * (3 * x * x - y * y), c * x * y * z, e * y * (4 * z * z - x * x - y * y),
              f * z * (2 * z * z - 3 * x * x - 3 * y * y), e * x * (4 * z * z - x * x - y * y),
              g * z * (x * x - y * y), a * x * (x * x - 3 * y * y)]
    return torch.stack(b)


def _rotation(q):
    w, x, y, z = q / q.norm(dim=0, keepdim=True)
    return torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y),
                        2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x),
                        2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)]).reshape(3, 3, -1)


def _exact_view(leaves, cam, degree, rows=2048):
    """Per view and block of pixels: colour, and what the outputs need of the blend."""
    means, scales, quats, opacity, sh = leaves
    dev, f64 = means.device, torch.float64
    R = torch.tensor(cam.R, dtype=f64, device=dev)
    tv = torch.tensor(cam.t, dtype=f64, device=dev)
    t = R @ means + tv[:, None]
    keep = ((t[2] > 0.2) & (opacity >= 1.0 / 255.0)).nonzero()[:, 0]
    keep = keep[torch.sort(t[2].detach()[keep].float(), stable=True)[1]]
    t, Rq, s = t[:, keep], _rotation(quats[:, keep]), scales[:, keep]
    A = (R @ Rq.reshape(3, -1)).reshape(3, 3, -1) * s
    S = (A[:, None] * A[None]).sum(2)
    lim = 1.3 * cam.width / (2 * cam.fx), 1.3 * cam.height / (2 * cam.fy)
    xr, yr = (t[0] / t[2]).clamp(-lim[0], lim[0]), (t[1] / t[2]).clamp(-lim[1], lim[1])
    J0 = torch.stack([cam.fx / t[2], torch.zeros_like(xr), -cam.fx * xr / t[2]])
    J1 = torch.stack([torch.zeros_like(yr), cam.fy / t[2], -cam.fy * yr / t[2]])
    SJ0, SJ1 = (S * J0).sum(1), (S * J1).sum(1)
    s00, s01, s11 = (J0 * SJ0).sum(0) + 0.3, (J0 * SJ1).sum(0), (J1 * SJ1).sum(0) + 0.3
    det = s00 * s11 - s01 * s01
    u, v = cam.fx * t[0] / t[2] + cam.cx, cam.fy * t[1] / t[2] + cam.cy
    centre = -(R.T @ tv)
    d = means[:, keep] - centre[:, None]
    K = (degree + 1) ** 2
    rgb = (0.5 + (sh[:K, :, keep] * _sh_basis(d / d.norm(dim=0), degree)[:, None]).sum(0)).clamp(min=0)
    P = cam.width * cam.height
    for p0 in range(0, P, rows):
        p = torch.arange(p0, min(P, p0 + rows), device=dev)
        px, py = (p % cam.width).double() + 0.5, (p // cam.width).double() + 0.5
        dx, dy = px[:, None] - u, py[:, None] - v
        g = opacity[keep] * torch.exp(-0.5 * (s11 * dx * dx - 2 * s01 * dx * dy + s00 * dy * dy) / det)
        ok = g >= 1.0 / 255.0
        a = torch.where(ok, g.clamp(max=0.99), 0.0)
        T = torch.cumprod(1 - a, 1)
        inc = ok & (T.detach() >= 1e-4)
        a = torch.where(inc, a, 0.0)
        T = torch.cumprod(1 - a, 1)
        w = a * torch.cat([torch.ones_like(T[:, :1]), T[:, :-1]], 1)
        tfin = T[:, -1] if T.shape[1] else torch.ones_like(px)
        yield keep, Rq, s, centre, R, (px, py, (w @ rgb.T).T, w, tfin)


def _exact_render(case, s, leaves, dl=None, accumulate=False):
    """Outputs of a render in float64 and, with dl, its parameter gradients."""
    n = case["gaussians"]
    color, depth, tfin, hits = [], [], [], []
    imp, wmax = torch.zeros(n, dtype=torch.float64, device="cuda"), torch.zeros(n, dtype=torch.float64, device="cuda")
    grads = [torch.zeros_like(x) for x in leaves]
    at = 0
    for cam in s["cams"]:
        P, P0 = cam.width * cam.height, 0
        for k, (keep, Rq, sc, centre, R, (px, py, c, w, T)) in enumerate(_exact_view(leaves, cam, case["degree"])):
            m = c.shape[1]
            if dl is not None and c.requires_grad:
                got = torch.autograd.grad(c, leaves, dl[:, at + P0: at + P0 + m], retain_graph=True, allow_unused=True)
                grads = [a + b if b is not None else a for a, b in zip(grads, got)]
            with torch.no_grad():
                best, j = (w.max(1) if w.shape[1] else (torch.zeros_like(T), torch.zeros_like(T, dtype=torch.long)))
                ray = torch.stack([(px - cam.cx) / cam.fx, (py - cam.cy) / cam.fy, torch.ones_like(px)])
                ray = R.T @ ray
                o = centre[:, None] - leaves[0][:, keep][:, j]
                Q = Rq[:, :, j] / sc[:, j]
                oo, dd = (Q * o[:, None]).sum(0), (Q * ray[:, None]).sum(0)
                depth.append(torch.where(best > 0, -(oo * dd).sum(0) / (dd * dd).sum(0), 0.0))
                imp.index_add_(0, keep, w.sum(0))
                wmax[keep] = torch.maximum(wmax[keep], w.max(0)[0])
                color.append(c.detach())
                tfin.append(T.detach())
            P0 += m
        at += P
    return torch.cat(color, 1), torch.cat(depth), torch.cat(tfin), imp, wmax, grads


def exact(case, seed):
    if case["kind"] == "criteria":
        return _exact_criteria(case, seed)
    if case["kind"] == "densify":
        return _exact_densify(case, seed)
    pixels = case["views"] * case["width"] * case["height"]
    if not case["width"] or case["gaussians"] * pixels > EXACT_PAIRS:
        return None
    s = prepare(case, seed)
    sc = s["scene"]
    leaves = [t.detach().double() for t in (sc.means, sc.scales, sc.quats, sc.opacity, sc.sh)]
    if case["kind"] == "render":
        color, depth, tfin, _, _, _ = _exact_render(case, s, leaves)
        return dict(color=color, depth=depth, imax=None, t_final=tfin)
    leaves = [t.requires_grad_() for t in leaves]
    out = {}
    if case["kind"] == "step":
        dl = s["dl"].double()
    else:
        # the loss gradient's sign comes from the colour itself
        with torch.no_grad():
            color = _exact_render(case, s, [t.detach() for t in leaves])[0]
        diff = color - s["target"].double()
        dl = torch.sign(diff) / diff.numel()
        out["loss"] = diff.abs().mean().reshape(1)
    color, depth, tfin, imp, wmax, grads = _exact_render(case, s, leaves, dl)
    if s["active"] is not None:
        grads = [g * (s["active"] != 0) for g in grads]
    out.update(color=color, depth=depth, imax=None)
    if case["kind"] == "loop":
        out.update(t_final=tfin, last=None, n_contrib=None, hit=None, importance=imp, wmax=wmax, area=None)
    out.update({"d_" + k: g for k, g in zip(GRADS, grads)})
    return out


def _exact_criteria(case, seed):
    s = prepare(case, seed)

    def mass(values):
        """The value whose descending prefix sum is nearest to 0.99 of the total."""
        x = torch.sort(values.double(), descending=True)[0]
        c = torch.cumsum(x, 0)
        return x[torch.argmin((c - 0.99 * c[-1]).abs())]

    tau = torch.stack([mass(v[v > 0]) for v in s["importance"]])
    return dict(visible=None, tau=tau, critical=None, critical_tau=mass(s["wmax"][s["area"] > 0]).reshape(1), blur=None,
                keep=None, count=None)


def _exact_densify(case, seed):
    s = prepare(case, seed)
    sc, n = s["scene"], case["gaussians"]
    hot = s["norm"].double() / s["count"].double() >= THRESHOLD
    big = sc.scales.max(0)[0].double() > SCALE_THRESHOLD
    clone, split = hot & ~big, hot & big
    p = [t.double() for t in (sc.means, sc.scales, sc.quats, sc.opacity[None], sc.sh.reshape(48, n))]
    a = p[3]
    a2 = 1 - torch.sqrt(1 - a)
    p[1] = torch.where(clone, p[1] * (a / (2 * a2 - a2 * a2 / math.sqrt(2.0))), p[1])
    p[3] = torch.where(clone, a2, a)
    p = [torch.cat([t, t[:, clone]], 1).float().double() for t in p]
    split = torch.nn.functional.pad(split, (0, p[0].shape[1] - n))
    m = p[0].shape[1]
    stay = [t[:, ~split] for t in p]
    half = [t[:, split].repeat_interleave(2, 1) for t in p]
    z = s["normals"][:, :, :m][:, :, split].double().permute(1, 2, 0).reshape(3, -1)
    half[0] = half[0] + (_rotation(half[2]) * (half[1] * z)[None]).sum(1)
    half[1] = half[1] / 1.6
    p = [torch.cat(t, 1).float() for t in zip(stay, half)]
    lo, hi = p[0].min(1, keepdim=True)[0], p[0].max(1, keepdim=True)[0]
    cell = ((p[0] - lo) * (1024.0 / (hi - lo))).clamp(max=1023.0).long()
    code = torch.zeros_like(cell[0])
    for b in range(10):
        for axis in range(3):
            code |= ((cell[axis] >> b) & 1) << (3 * b + 2 - axis)
    order = torch.sort(code, stable=True)[1]
    p = [t[:, order].double() for t in p]
    return dict(means=p[0], scales=p[1], quats=p[2], opacity=p[3][0], sh=p[4].reshape(16, 3, -1), perm=None,
                cloned=None, halved=None)
