"""The compositing render kernels at the sizes where their branches change:
both lane layouts of the backward (few tiles: four wavefronts a tile; many:
one), culling of needle-shaped and sub-pixel ellipses against quadrants and
row bands, opacities on both sides of the alpha clamp, and stacks deep enough
that the transmittance leaves the range in which its scale factor is skipped.
Against the FP64 oracle at the compositing bar (scaled error <= 1e-5)."""
import numpy as np
import pytest
import torch

import paper_2606_09794_amd as P
import workloads as W
from gpu_util import compare
from oracle import raster_ref as RR

pytestmark = pytest.mark.gpu
TOL = 1e-5
WIN = (70, 45)          # the window that holds every primitive


def _scene(kind):
    w, h = WIN
    rng = np.random.default_rng(sum(map(ord, kind)))
    if kind == "needles":       # 3 sigma from a hundredth of a pixel to the whole window
        sc = W.draw_splat_scene(60, 500, w, h, scale=(2e-4, 1.0))
        sc.scales[:, 2] = sc.scales[:, 0]
    elif kind == "opacities":
        sc = W.draw_splat_scene(61, 300, w, h, scale=(0.05, 0.4))
        sc.opac[:] = rng.choice([0.0, 1e-30, 1e-6, 0.3, 0.98, 0.99, 0.995, 1.0, 3.0, 127.0, 500.0],
                                sc.n).astype(np.float32)
    else:                       # "deep": over 200 clamped layers, T below 2^-500
        sc = W.draw_splat_scene(62, 500, w, h, scale=(1.0, 3.0), depth=(3.0, 6.0), behind=0.0,
                                opac=(0.9, 1.0))
    return sc


@pytest.mark.parametrize("canvas", [WIN, (896, 896)], ids=["few-tiles", "many-tiles"])
@pytest.mark.parametrize("kind", ["needles", "opacities", "deep"])
def test_render_branches(kind, canvas):
    w, h = WIN
    sc = _scene(kind)
    x0, y0 = ((canvas[0] - w) // 2 // 16 * 16, (canvas[1] - h) // 2 // 16 * 16)
    cam = P.Camera(sc.cam["R"], sc.cam["t"], sc.cam["fx"], sc.cam["fy"], sc.cam["cx"] + x0,
                   sc.cam["cy"] + y0, *canvas)
    d = [torch.from_numpy(np.ascontiguousarray(x)).cuda()
         for x in (sc.means, sc.scales, sc.rots, sc.opac, sc.colors)]
    g = torch.zeros((canvas[1], canvas[0], 3), device="cuda")
    g[y0:y0 + h, x0:x0 + w] = torch.from_numpy(sc.grad_image).cuda()
    img, ws = P.raster_fwd(*d, cam, 1024)
    out = P.raster_bwd(*d, cam, ws, g, 1024, geometry=True)
    two = P.raster_bwd(*d, cam, ws, g, 1024)
    torch.cuda.synchronize()
    ref, scale = RR.render(sc.means, sc.scales, sc.rots, sc.opac, sc.colors, sc.cam,
                           grad_image=sc.grad_image, geometry=True)
    compare(img[y0:y0 + h, x0:x0 + w].cpu().numpy(), ref["image"], scale["image"], "image", TOL)
    for name, v in zip(("colors", "opac", "means", "scales", "rots"), out):
        compare(v.cpu().numpy(), ref[name], scale[name], f"grad {name}", TOL)
    for name, v in zip(("colors", "opac"), two):
        compare(v.cpu().numpy(), ref[name], scale[name], f"grad {name} alone", TOL)


@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_unbounded_opacity_composites_at_the_clamp(value):
    """An infinite opacity, or a NaN (which the clamp's minimum drops), acts as
    any opacity that is clamped on its whole support."""
    sc = _scene("opacities")
    res = []
    for v in (value, 500.0):
        op = np.where(sc.opac == 500.0, np.float32(v), sc.opac)
        d = [torch.from_numpy(np.ascontiguousarray(x)).cuda()
             for x in (sc.means, sc.scales, sc.rots, op, sc.colors)]
        cam = P.Camera(sc.cam["R"], sc.cam["t"], sc.cam["fx"], sc.cam["fy"], sc.cam["cx"],
                       sc.cam["cy"], *WIN)
        img, ws = P.raster_fwd(*d, cam, 1024)
        res.append((img, *P.raster_bwd(*d, cam, ws, torch.from_numpy(sc.grad_image).cuda(), 1024)))
    assert torch.equal(res[0][0], res[1][0])
    for x, y in zip(res[0][1:], res[1][1:]):
        assert torch.allclose(x, y, rtol=1e-6, atol=1e-9)


@pytest.mark.parametrize("n", [2, 63, 255, 256, 257, 1024, 1025])
def test_list_lengths_with_equal_depths(n):
    """One tile that every primitive reaches, at the lengths where the sort
    and the binning chunks change, with exact depth ties and depths that are
    equal only in float32 (the camera is turned by 1e-6 rad)."""
    rng = np.random.default_rng(70 + n)
    th = 1e-6
    R = np.array([[np.cos(th), 0.0, np.sin(th)], [0.0, 1.0, 0.0], [-np.sin(th), 0.0, np.cos(th)]])
    cam = dict(R=R, t=np.zeros(3), fx=20.0, fy=20.0, cx=8.0, cy=8.0, width=16, height=16)
    x = rng.uniform(-0.5, 0.5, n)
    x[: n // 2] = rng.choice(x[n // 2:], n // 2)
    z = np.where(rng.random(n) < 0.3, 4.0, rng.uniform(3.0, 6.0, n))
    sc = W.SplatScene(means=np.stack([x, rng.uniform(-0.5, 0.5, n), z], -1).astype(np.float32),
                      scales=np.exp(rng.uniform(np.log(0.3), np.log(0.6), (n, 3))).astype(np.float32),
                      rots=rng.standard_normal((n, 4)).astype(np.float32),
                      opac=rng.uniform(0.02, 0.2, n).astype(np.float32),
                      colors=rng.standard_normal((n, 3)).astype(np.float32),
                      grad_image=rng.standard_normal((16, 16, 3)).astype(np.float32), cam=cam)
    d = [torch.from_numpy(np.ascontiguousarray(v)).cuda()
         for v in (sc.means, sc.scales, sc.rots, sc.opac, sc.colors)]
    c = P.Camera(R, cam["t"], 20.0, 20.0, 8.0, 8.0, 16, 16)
    img, ws = P.raster_fwd(*d, c, 2048)
    out = P.raster_bwd(*d, c, ws, torch.from_numpy(sc.grad_image).cuda(), 2048, geometry=True)
    ref, scale = RR.render(sc.means, sc.scales, sc.rots, sc.opac, sc.colors, cam,
                           grad_image=sc.grad_image, geometry=True)
    compare(img.cpu().numpy(), ref["image"], scale["image"], "image", TOL)
    for name, v in zip(("colors", "opac", "means", "scales", "rots"), out):
        compare(v.cpu().numpy(), ref[name], scale[name], f"grad {name}", TOL)


def test_camera_centre_on_the_device_equals_the_host():
    """The centre written by a kernel is the float32 of the host's FP64 one; a
    side stream gets it on that stream. FP64 sums of three products in two
    orders differ by less than 4 * 2^-53 of the terms, float32 rounds to 2^-24."""
    rng = np.random.default_rng(5)
    side = torch.cuda.Stream()
    for i in range(64):
        rot, _ = np.linalg.qr(rng.standard_normal((3, 3)))
        t = rng.standard_normal(3) * 10.0 ** rng.integers(-2, 3)
        cam = P.Camera(rot, t, 100.0, 100.0, 8.0, 8.0, 16, 16)
        host = cam.centre("cpu").numpy()
        with torch.cuda.stream(side if i % 2 else torch.cuda.current_stream()):
            got = cam.centre("cuda").cpu().numpy()
        assert got.shape == (1, 3) and got.dtype == np.float32
        tol = 2.0 ** -23 * np.abs(host) + 2.0 ** -51 * np.abs(t).sum()
        assert np.all(np.abs(got - host) <= tol), (i, got, host)


@pytest.mark.parametrize("canvas", [(16, 16), (896, 896)], ids=["few-tiles", "many-tiles"])
def test_infinite_colour_behind(canvas):
    """An infinite colour (an overflow of the appearance): the entry in front of it
    gets an infinite opacity gradient of the sign that c - R has, R the colour seen
    behind it, its own the other sign, and those behind it what they get beside a
    finite colour, bit for bit. (From the next entry on R itself is inf - inf.)"""
    cam = P.Camera(np.eye(3), np.zeros(3), 20.0, 20.0, canvas[0] / 2, canvas[1] / 2, *canvas)
    n = 5
    means = torch.tensor([[0.0, 0.0, 3.0 + i] for i in range(n)], device="cuda")
    scales = torch.full((n, 3), 0.4, device="cuda")
    rots = torch.tensor([[1.0, 0.0, 0.0, 0.0]] * n, device="cuda")
    opac = torch.tensor([0.2, 0.3, 0.4, 0.5, 0.6], device="cuda")
    g = torch.ones((canvas[1], canvas[0], 3), device="cuda")
    grads = []
    for c in (float("inf"), 1.0):
        col = torch.full((n, 3), 0.5, device="cuda")
        col[2, 1] = c
        img, ws = P.raster_fwd(means, scales, rots, opac, col, cam, 64)
        grads.append([x.cpu() for x in P.raster_bwd(means, scales, rots, opac, col, cam, ws, g, 64)])
    go = grads[0][1]
    assert go[1] == -float("inf") and go[2] == float("inf"), go
    assert torch.equal(go[3:], grads[1][1][3:])
    assert torch.equal(grads[0][0], grads[1][0])      # the colours' gradients do not hold colours


def test_camera_centre_is_there_for_every_stream():
    """The centre of a camera made on a busy stream is read by another one at once,
    without an event between them."""
    busy = torch.randn((8192, 8192), device="cuda")
    side = torch.cuda.Stream()
    torch.cuda.synchronize()
    for i in range(4):
        cam = P.Camera(np.eye(3), [1.0 + i, -2.0, 3.0], 100.0, 100.0, 8.0, 8.0, 16, 16)
        for _ in range(8):
            busy = (busy @ busy) * 1e-4
        c = cam.centre("cuda")
        with torch.cuda.stream(side):
            got = c.clone()
        side.synchronize()
        assert torch.equal(got.cpu(), torch.tensor([[-1.0 - i, 2.0, -3.0]])), i
    torch.cuda.synchronize()


def test_view_of_a_camera_with_its_own_centre():
    """A camera class that says its centre differently is asked for it."""
    class Shifted(P.Camera):
        def centre(self, device):
            return super().centre(device) + 0.5

    sc = W.draw_splat_scene(64, 200, 48, 32)
    w = W.draw_workload(64, 200, 2, 1, with_sh=False)
    lob = [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (w.quat, w.shape, w.rgbw, w.c0)]
    d = [torch.from_numpy(np.ascontiguousarray(x)).cuda() for x in (sc.means, sc.scales, sc.rots, sc.opac)]
    args = (sc.cam["R"], sc.cam["t"], sc.cam["fx"], sc.cam["fy"], sc.cam["cx"], sc.cam["cy"], 48, 32)
    cam = Shifted(*args)
    got = P.render_view(*lob, *d, cam, tile_capacity=512)
    rgb = P.nasg_eval_fwd(*lob, means=d[0], cams=P.Camera(*args).centre("cuda") + 0.5)
    assert torch.equal(got, P.raster_fwd(*d, rgb[0].contiguous(), cam, 512)[0])
