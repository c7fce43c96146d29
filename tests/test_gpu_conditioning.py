"""Gradients where two large terms nearly cancel, or where 1 - (d.z)^2 leaves the
range that a rounding error of d.z allows, against the FP64 oracle."""
import numpy as np
import pytest
import torch

import paper_2606_09794_amd as P
import workloads as W
from gpu_util import compare, dgeo, oracle_nasg, upload
from oracle import nasg_ref as R

pytestmark = pytest.mark.gpu
TOL = 1e-5


def _run(w, norm="exact"):
    d = upload(w)
    rgb = P.nasg_eval_fwd(d["quat"], d["shape"], d["rgbw"], d["c0"], norm=norm, **dgeo(d))
    fused = torch.empty_like(rgb)
    g = P.nasg_eval_bwd(d["quat"], d["shape"], d["rgbw"], d["c0"], d["grad_rgb"], norm=norm,
                        rgb_out=fused, **dgeo(d))
    torch.cuda.synchronize()
    return rgb.cpu().numpy(), fused.cpu().numpy(), {k: x.cpu().numpy() for k, x in g.items()}


@pytest.mark.parametrize("v", [1, 2, 5, 16])
def test_zeta_gradient_next_to_the_carrier_zero(v):
    """EXACT normaliser, zeta next to pi, a slow carrier: d ln N / d zeta and
    d ln c / d zeta are both about 2/(pi - zeta) with opposite signs. With t =
    tan(zeta/2), c = cos^2(theta/2), d ln N / d zeta = t (1 - (1 - Psi)/B) is
    rearranged into two terms that do not cancel,
        N p E (t c - sin(theta)/2) = -N p E cos(theta/2) sin(k d.x/2)/cos(zeta/2)
    and -G t (1 - Psi)/B, each held to the parity bar; of the terms before the
    rearrangement 3e-8 may be left (sine and cosine of the half phase to about 1e-8,
    entering t c and sin(theta)/2 three times in all; formed in float32 they leave
    several 1e-7)."""
    n, k = 3000, 4
    w = W.draw_workload(50 + v, n, k, v, with_sh=False)
    rng = np.random.default_rng(v)
    off = np.exp(rng.uniform(np.log(0.01), np.log(1.0), (k, n))) * rng.choice([-1.0, 1.0], (k, n))
    w.shape[..., 3] = np.pi * rng.choice([-1.0, 1.0, 3.0], (k, n)) + off
    w.shape[..., 2] = np.exp(rng.uniform(np.log(1e-3), 0.0, (k, n)))
    _, _, g = _run(w)
    ref, scale = oracle_nasg(w, "exact")
    ax, _, az = R.frame_from_quat(w.quat)
    dirs, _ = R.view_directions(w.means, w.cams)
    lam, a, kk, zeta = np.moveaxis(w.shape.astype(np.float64), -1, 0)
    t = R.lobe_terms(dirs, ax, az, w.shape, R.norm_exact(lam, a, kk, zeta)[0])
    psi, _, _, om = R.psi(lam * (1.0 + a), kk)
    tz = np.tan(zeta / 2)
    B = psi * 2.0 * np.cos(zeta / 2) ** 2 + om
    weight = np.abs(w.grad_rgb[None] * np.transpose(w.rgbw, (0, 2, 1))[:, None]).sum(-1)   # [K][V][N]
    first = np.abs(t["p"] * t["E"] * t["Cn"] * np.cos(t["arg"] / 2) * np.sin(kk * t["dx"].swapaxes(0, 1) / 2).swapaxes(0, 1)
                   / np.cos(zeta / 2)[:, None])
    second = np.abs(t["G"] * (tz * om / B)[:, None])
    bar = TOL * (weight * (first + second)).sum(1) + 3e-8 * scale["shape"][..., 3]
    err = np.abs(g["shape"][..., 3] - ref["shape"][..., 3])
    worst = float((err / (bar + 1e-30)).max())
    print(f"zeta error over its bar: {worst:.3g}; norm {np.linalg.norm(err) / np.linalg.norm(ref['shape'][..., 3]):.2g}")
    assert worst <= 1.0
    for name in ("quat", "shape", "rgbw", "c0", "geom"):
        compare(g[name], ref[name], scale[name], name, TOL)


def _check(w, norm="exact"):
    rgb, fused, g = _run(w, norm)
    ref, scale = oracle_nasg(w, norm)
    compare(rgb, ref["rgb"], scale["rgb"], "rgb", TOL)
    compare(fused, ref["rgb"], scale["rgb"], "rgb (fused)", TOL)
    for name, x in g.items():
        compare(x, ref[name], scale[name], name, TOL)


@pytest.mark.parametrize("norm", ["exact", "approx"])
def test_gradients_next_to_the_axis(norm):
    """Directions 1e-10 to 1e-7 off the lobe axis, where q = |d + z|^2 rounds to 4
    or above: ln kappa/(1 - (d.z)^2) -> -1/4 there, with d.x up to the offset and
    tau up to a, so nothing that multiplies it vanishes."""
    offs = [0.0, 1e-10, 1e-9, 5e-9, 1e-8, 1.4e-8, 2e-8, 3e-8, 6e-8, 1e-7]
    dirs = [(e * c, e * s, 1.0) for e in offs for c, s in ((1, 0), (1, 1), (0, 1))]
    lobes = [(lam, a, k) for lam in (0.3, 1.0, 30.0, 1000.0) for a in (0.0, 1.0, 1000.0) for k in (0.0, 8.0)]
    n = len(dirs) * len(lobes)
    w = W.draw_workload(3, n, 1, 1, dirs_mode=True, with_sh=False)
    w.quat[...] = (1.0, 0.0, 0.0, 0.0)
    w.dirs[...] = np.repeat(np.array(dirs, np.float32), len(lobes), axis=0)
    w.shape[0, :, :3] = np.tile(np.array(lobes, np.float32), (len(dirs), 1))
    _check(w, norm)


@pytest.mark.parametrize("k,v", [(1, 1), (8, 3), (8, 16)])
def test_frames_aimed_at_a_camera(k, v):
    """Float32 frames whose axis is the direction to one of the cameras as nearly
    as float32 quaternions give it: that view's terms meet the other views' and
    the other lobes' in one sum."""
    n = 4000
    w = W.draw_workload(70 + v, n, k, v, with_sh=False)
    rng = np.random.default_rng(v)
    d, _ = R.view_directions(w.means, w.cams)
    for lobe in range(k):
        z = d[lobe % v]                                   # [N][3]
        up = np.cross(z, rng.normal(size=(n, 3)))
        x = up / np.linalg.norm(up, axis=-1, keepdims=True)
        y = np.cross(z, x)
        m = np.stack([x, y, z], -1)                       # columns
        t = np.trace(m, axis1=1, axis2=2)
        q = np.stack([1.0 + t, m[:, 2, 1] - m[:, 1, 2], m[:, 0, 2] - m[:, 2, 0],
                      m[:, 1, 0] - m[:, 0, 1]], -1)
        w.quat[lobe] = q / np.linalg.norm(q, axis=-1, keepdims=True)
    _check(w)


@pytest.mark.parametrize("norm", ["exact", "approx"])
def test_next_to_the_antipode(norm):
    """Directions 1e-30 to 1e-6 off -z with an exact frame: G = N e^{-2 lam (1 - E
    kappa)} kappa^tau, tau = a cos^2(phi), keeps its limit (N e^{-2 lam} along y, 0
    elsewhere unless a is small) however small kappa = |d + z|^2/4 > 0 is. The
    gradients, which hold 1/kappa, are compared where those are in FP32's range
    and are finite everywhere."""
    offs = [0.0, 1e-30, 1e-20, 1e-18, 1e-17, 1e-16, 1e-15, 1e-14, 1e-12, 1e-9, 1e-6]
    phis = [(1, 0), (0, 1), (1, 1), (0.01, 1)]
    dirs = np.array([(e * c, e * s, -1.0) for e in offs for c, s in phis], np.float32)
    lobes = [(lam, a, k) for lam in (0.05, 0.5, 3.0) for a in (0.0, 1e-3, 0.1, 10.0) for k in (0.0, 3.0)]
    n = len(dirs) * len(lobes)
    w = W.draw_workload(4, n, 1, 1, dirs_mode=True, with_sh=False)
    w.quat[...] = (1.0, 0.0, 0.0, 0.0)
    w.dirs[...] = np.repeat(dirs, len(lobes), axis=0)
    w.shape[0, :, :3] = np.tile(np.array(lobes, np.float32), (len(dirs), 1))
    rgb, fused, g = _run(w, norm)
    ref, scale = oracle_nasg(w, norm)
    compare(rgb, ref["rgb"], scale["rgb"], "rgb", TOL)
    compare(fused, ref["rgb"], scale["rgb"], "rgb (fused)", TOL)
    far = np.abs(w.dirs[:, :2]).max(-1) > 5e-15
    for name, x in g.items():
        assert np.isfinite(x).all(), name
        at = (np.s_[:, far] if name in ("quat", "shape") else np.s_[:, :, far] if name == "rgbw" else np.s_[far])
        compare(x[at], ref[name][at], scale[name][at], name, TOL)
