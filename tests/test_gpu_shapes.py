"""The built-in launch shapes: on both sides of every line of the choice by N,
K and V, the colours and gradients equal those of the one-lane mapping up to
the order of the lobe and view sums (a few float32 roundings of terms whose
absolute sum the oracle's scale measures; checked against the oracle at the
bar of the lane-mapping tests)."""
import numpy as np
import pytest
import torch

import paper_2606_09794_amd as P
import workloads as W
from gpu_util import compare, oracle_nasg, oracle_sh, upload

pytestmark = pytest.mark.gpu
TOL = 1e-5


def _take(w, m=96):
    idx = np.unique(np.concatenate([np.arange(m // 2), w.n - 1 - np.arange(m // 2)]) % w.n)
    return idx, W.take_primitives(w, idx)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("n", [1, 4097, 16385, 32769])
@pytest.mark.parametrize("k,v", [(1, 1), (5, 1), (16, 1), (2, 2), (3, 2), (9, 2), (1, 4), (8, 3), (2, 7),
                                 (6, 6), (7, 8), (16, 5), (1, 9), (2, 18), (3, 17), (9, 17), (8, 20), (16, 33)])
def test_nasg_shapes(n, k, v, dtype):
    w = W.draw_workload(n + 64 * k + v, n, k, v, dtype=dtype, with_sh=False)
    d = upload(w)
    idx, sub = _take(w)
    ref, scale = oracle_nasg(sub, "exact")
    rgb = P.nasg_eval_fwd(d["quat"], d["shape"], d["rgbw"], d["c0"], means=d["means"], cams=d["cams"])
    fused = torch.full_like(rgb, float("nan"))
    g = P.nasg_eval_bwd(d["quat"], d["shape"], d["rgbw"], d["c0"], d["grad_rgb"], means=d["means"],
                        cams=d["cams"], rgb_out=fused)
    torch.cuda.synchronize()
    assert torch.isfinite(rgb).all() and torch.isfinite(fused).all()
    t = torch.from_numpy(idx).cuda()
    compare(rgb[:, t].cpu().numpy(), ref["rgb"], scale["rgb"], "rgb", TOL)
    compare(fused[:, t].cpu().numpy(), ref["rgb"], scale["rgb"], "fused rgb", TOL)
    for name, x in (("quat", g["quat"][:, t]), ("shape", g["shape"][:, t]),
                    ("rgbw", g["rgbw"][:, :, t]), ("c0", g["c0"][t]), ("geom", g["geom"][t])):
        compare(x.cpu().numpy(), ref[name], scale[name], name, TOL)


@pytest.mark.parametrize("n", [1, 4097, 8193, 16385, 36865, 45057, 73729, 131073])
@pytest.mark.parametrize("v", [1, 3, 7, 13, 16, 33])
def test_sh_shapes(n, v):
    w = W.draw_workload(n + v, n, 1, v)
    d = upload(w)
    idx, sub = _take(w)
    ref, scale = oracle_sh(sub)
    rgb = P.sh3_eval_fwd(d["sh"], means=d["means"], cams=d["cams"])
    g = P.sh3_eval_bwd(d["sh"], d["grad_rgb"], means=d["means"], cams=d["cams"])
    torch.cuda.synchronize()
    t = torch.from_numpy(idx).cuda()
    compare(rgb[:, t].cpu().numpy(), ref["rgb"], scale["rgb"], "rgb", TOL)
    compare(g["sh"][:, :, t].cpu().numpy(), ref["sh"], scale["sh"], "sh", TOL)
    compare(g["geom"][t].cpu().numpy(), ref["geom"], scale["geom"], "geom", TOL)


@pytest.mark.parametrize("family", ["nasg", "sg", "sb", "sc", "asg"])
@pytest.mark.parametrize("k,v", [(1, 17), (2, 9), (3, 8), (5, 20)])
def test_family_shapes(family, k, v):
    w = W.draw_workload(7 * k + v, 300, k, v, family=family, with_sh=False)
    d = upload(w)
    ref, scale = oracle_nasg(w, "exact")
    g = P.nasg_eval_bwd(d["quat"], d["shape"], d["rgbw"], d["c0"], d["grad_rgb"], means=d["means"],
                        cams=d["cams"], family=family)
    torch.cuda.synchronize()
    for name, x in g.items():
        compare(x.cpu().numpy(), ref[name], scale[name], name, TOL)


@pytest.mark.parametrize("sizes", [[(300, 8, 1), (5000, 4, 16), (0, 8, 4)], [(40_000, 4, 20)] * 3])
def test_batch_tiles_adapt(sizes):
    """A plan without a tile size cuts few scenes into small tiles, with the
    results of a plan of large tiles bit for bit."""
    plans = []
    for ti in (None, 8):
        scenes = []
        for s, (n, k, v) in enumerate(sizes):
            d = upload(W.draw_workload(90 + s, n, k, v, with_sh=False))
            d["grads"] = {q: t.fill_(float("nan")) for q, t in P.nasg_grad_buffers(k, n, "cuda").items()}
            d["rgb"] = torch.full((v, n, 3), float("nan"), device="cuda")
            scenes.append(d)
        plan = P.NasgBatchPlan(scenes, tile_iters=ti)
        plan.run()
        plans.append((plan, scenes))
    torch.cuda.synchronize()
    assert plans[0][0].n_items > plans[1][0].n_items
    for a, b in zip(plans[0][1], plans[1][1]):
        assert torch.equal(a["rgb"], b["rgb"])
        for q in a["grads"]:
            assert torch.equal(a["grads"][q], b["grads"][q])
            assert torch.isfinite(a["grads"][q]).all()


@pytest.mark.parametrize("n,k,v,param", [(24576, 1, 16, "quat"), (24577, 1, 16, "quat"),
                                         (98304, 2, 8, "quat"), (98305, 2, 8, "quat"),
                                         (196608, 2, 7, "angles"), (196609, 2, 7, "angles")])
def test_batch_follows_the_shape_by_n(n, k, v, param):
    """On both sides of the lines in N a scene in a batch equals its own launch
    bit for bit, beside a small scene of the same K and V."""
    scenes = []
    for m in (n, 700):
        w = W.draw_workload(m % 1000 + k, m, k, v, param=param, with_sh=False)
        d = upload(w)
        d["param"] = param
        d["grads"] = {q: t.fill_(float("nan")) for q, t in P.nasg_grad_buffers(k, m, "cuda").items()}
        d["rgb"] = torch.full((v, m, 3), float("nan"), device="cuda")
        scenes.append(d)
    P.NasgBatchPlan(scenes).run()
    for d in scenes:
        rgb = torch.empty_like(d["rgb"])
        g = P.nasg_eval_bwd(d["quat"], d["shape"], d["rgbw"], d["c0"], d["grad_rgb"], means=d["means"],
                            cams=d["cams"], param=param, rgb_out=rgb)
        fwd = P.nasg_eval_fwd(d["quat"], d["shape"], d["rgbw"], d["c0"], means=d["means"],
                              cams=d["cams"], param=param)
        torch.cuda.synchronize()
        assert torch.equal(d["rgb"], rgb) and torch.equal(rgb, fwd)
        for q in g:
            assert torch.equal(d["grads"][q], g[q]), q


@pytest.mark.parametrize("v", [1, 2, 4, 16])
def test_raw_activations_over_their_range(v):
    """The paper's raw values from denormal to saturated, on both sides of the
    exponential's reduction steps: called and inlined activations (by the views
    per lane and the direction) against the oracle at the same bar. The colours
    and the gradients of the weights and c0, whose terms stay in FP32's range: a
    weight of 1e-30 leaves the others' below it."""
    n, k = 1500, 8
    w = W.draw_workload(900 + v, n, k, v, param="angles", with_sh=False)
    rng = np.random.default_rng(v)
    step = 0.5 * np.log(2.0)
    edges = np.array([0.0, 1e-30, 1e-8, 1e-4, 0.5 * step, 0.999 * step, 1.001 * step, 3 * step, 1.0,
                      5.0, 18.0, 40.0, 380.0, 1e4])
    pick = lambda size: (rng.choice(edges, size) * rng.choice([-1.0, 1.0], size)).astype(np.float32)  # noqa: E731
    w.rgbw[:] = pick(w.rgbw.shape)
    w.shape[..., 2] = pick(w.shape.shape[:-1])
    w.quat[..., :3] = np.where(rng.random(w.quat[..., :3].shape) < 0.3,
                               np.clip(pick(w.quat[..., :3].shape), -5.0, 5.0), w.quat[..., :3])
    d = upload(w)
    rgb = P.nasg_eval_fwd(d["quat"], d["shape"], d["rgbw"], d["c0"], means=d["means"], cams=d["cams"],
                          param="angles")
    fused = torch.empty_like(rgb)
    g = P.nasg_eval_bwd(d["quat"], d["shape"], d["rgbw"], d["c0"], d["grad_rgb"], means=d["means"],
                        cams=d["cams"], param="angles", rgb_out=fused)
    ref, scale = oracle_nasg(w, "exact")
    compare(rgb.cpu().numpy(), ref["rgb"], scale["rgb"], "rgb", TOL)
    compare(fused.cpu().numpy(), ref["rgb"], scale["rgb"], "rgb (fused)", TOL)
    for name in ("rgbw", "c0"):
        compare(g[name].cpu().numpy(), ref[name], scale[name], name, TOL)


def test_raw_weights_are_rounded_once():
    """A raw weight's tanh is formed in FP64 and rounded to float32 once: of a million
    colours w G, G known from a saturated weight, the FP64 tanh rounded explains all
    but those whose tanh lies within 2e-14 (its FP64 error at |u| >= 0.01) of the
    middle between two float32 values: an expected 0.3 at most, 4 allowed."""
    n = 1 << 20
    w = W.draw_workload(77, n, 1, 1, param="angles", dirs_mode=True, with_sh=False)
    rng = np.random.default_rng(77)
    w.rgbw[:] = np.exp(rng.uniform(np.log(0.01), np.log(8.0), w.rgbw.shape)) * rng.choice([-1.0, 1.0], w.rgbw.shape)
    w.shape[..., :2] = 0.0             # lam = a = 1: no G near float32's smallest
    w.c0[:] = 0.0
    d = upload(w)
    one = torch.full_like(d["rgbw"], 30.0)
    G = P.nasg_eval_fwd(d["quat"], d["shape"], one, d["c0"], dirs=d["dirs"], param="angles")
    got = P.nasg_eval_fwd(d["quat"], d["shape"], d["rgbw"], d["c0"], dirs=d["dirs"], param="angles")
    want = torch.tanh(d["rgbw"][0].double()).float().T * G[0]
    off = int((got[0] != want).sum())
    print(f"{off} of {3 * n} colours differ")
    assert off <= 4


@pytest.mark.parametrize("v", [1, 2, 4, 16])
def test_raw_gradients_at_the_reduction_steps(v):
    """The gradients that the activations' exponentials feed (shape and quat among
    them), with the raw bandwidths, frequency and frame on both sides of the
    exponentials' reduction steps and at saturation, and ordinary weights."""
    n, k = 1500, 8
    w = W.draw_workload(950 + v, n, k, v, param="angles", with_sh=False)
    rng = np.random.default_rng(v)
    step = 0.5 * np.log(2.0)
    edges = np.array([0.0, 1e-8, 1e-4, 0.5 * step, 0.999 * step, 1.001 * step, 2.999 * step, 3.001 * step, 1.0, 5.0])
    pick = lambda size, more=(): (rng.choice(np.append(edges, more), size)  # noqa: E731
                                  * rng.choice([-1.0, 1.0], size)).astype(np.float32)
    w.shape[..., :2] = np.where(rng.random(w.shape[..., :2].shape) < 0.5, pick(w.shape[..., :2].shape), w.shape[..., :2])
    w.shape[..., 2] = pick(w.shape.shape[:-1], (18.0, 380.0))
    w.quat[..., :3] = np.where(rng.random(w.quat[..., :3].shape) < 0.3, pick(w.quat[..., :3].shape, (18.0,)),
                               w.quat[..., :3])
    d = upload(w)
    fused = torch.empty((v, n, 3), device="cuda")
    g = P.nasg_eval_bwd(d["quat"], d["shape"], d["rgbw"], d["c0"], d["grad_rgb"], means=d["means"],
                        cams=d["cams"], param="angles", rgb_out=fused)
    ref, scale = oracle_nasg(w, "exact")
    compare(fused.cpu().numpy(), ref["rgb"], scale["rgb"], "rgb", TOL)
    for name, x in g.items():
        compare(x.cpu().numpy(), ref[name], scale[name], name, TOL)


@pytest.mark.parametrize("lanes,vpl", [(4, 1), (8, 1), (16, 1), (8, 2), (8, 4)])
@pytest.mark.parametrize("k", [1, 3, 8, 13])
def test_broadcast_forward_has_the_one_lane_bits(k, lanes, vpl):
    """Each broadcast mapping's colours equal those of one lane per primitive with
    the same views per lane bit for bit, also with lanes left without a lobe."""
    n, v = 700, vpl + 1
    d = upload(W.draw_workload(31 * k + lanes, n, k, v, with_sh=False))
    got = []
    try:
        for m in ((lanes, vpl, 256, 1), (1, vpl, 256, 0)):
            P.set_tuning(0, k, v, 0, *m)
            got.append(P.nasg_eval_fwd(d["quat"], d["shape"], d["rgbw"], d["c0"], means=d["means"], cams=d["cams"]))
    finally:
        P.set_tuning(0, k, v, 0, 0, 0)
    torch.cuda.synchronize()
    assert torch.equal(*got)


def _graph(fn):
    """Four calls of fn, captured; the graph keeps fn, and so the tensors it holds."""
    s, g = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        fn()
        s.synchronize()
        with torch.cuda.graph(g, stream=s):
            for _ in range(4):
                fn()
    g.fn = fn
    return g


def _device_us(*graphs):
    """Device time of a call of each: the fastest of many replays, in turn."""
    a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
    best = [float("inf")] * len(graphs)
    for _ in range(100):
        for i, g in enumerate(graphs):
            a.record()
            g.replay()
            b.record()
            b.synchronize()
            best[i] = min(best[i], 250.0 * a.elapsed_time(b))
    return best


def _bwd_graph(w):
    d = upload(w)
    grads = P.nasg_grad_buffers(w.k, w.n, "cuda")
    return _graph(lambda: P.nasg_eval_bwd(
        d["quat"], d["shape"], d["rgbw"], d["c0"], d["grad_rgb"], means=d["means"], cams=d["cams"],
        param=w.param, family=w.family, grads=grads))


@pytest.mark.parametrize("family", ["nasg", "sg", "asg"])
@pytest.mark.parametrize("k,v", [(1, 7), (1, 16), (2, 16), (1, 24)])
def test_few_lobes_take_no_longer_than_eight(family, k, v):
    """Few primitives need the lanes however few lobes they have: a backward of
    one or two lobes (two to three and a half times that of eight, where its lanes
    followed the lobes at any N) against that of eight, with a third for noise."""
    us = _device_us(*[_bwd_graph(W.draw_workload(5, 4096, lobes, v, family=family, with_sh=False))
                      for lobes in (k, 8)])
    assert us[0] <= 1.33 * us[1], us


@pytest.mark.parametrize("family", ["nasg", "asg"])
@pytest.mark.parametrize("n,k,v", [(8192, 4, 9), (8193, 4, 9), (8193, 5, 9), (40960, 2, 5), (40961, 2, 5),
                                   (40961, 1, 17), (40961, 3, 16), (131073, 1, 5)])
def test_family_shapes(family, n, k, v):
    w = W.draw_workload(n + k, n, k, v, family=family, with_sh=False)
    d = upload(w)
    idx, sub = _take(w)
    ref, scale = oracle_nasg(sub, "exact")
    kw = dict(means=d["means"], cams=d["cams"], family=family)
    rgb = P.nasg_eval_fwd(d["quat"], d["shape"], d["rgbw"], d["c0"], **kw)
    g = P.nasg_eval_bwd(d["quat"], d["shape"], d["rgbw"], d["c0"], d["grad_rgb"], **kw)
    torch.cuda.synchronize()
    t = torch.from_numpy(idx).cuda()
    for name, x in (("rgb", rgb[:, t]), ("quat", g["quat"][:, t]), ("shape", g["shape"][:, t]),
                    ("rgbw", g["rgbw"][:, :, t]), ("c0", g["c0"][t]), ("geom", g["geom"][t])):
        compare(x.cpu().numpy(), ref[name], scale[name], name, TOL)


@pytest.mark.parametrize("n,v,param", [(4096, 7, "quat"), (4096, 8, "angles"), (30000, 16, "quat"),
                                       (30000, 16, "angles")])
def test_one_lobe_keeps_four_lanes_for_few_primitives(n, v, param):
    """The built-in choice against four lanes per primitive, which take 0.5 to
    0.8 of one lane's time here; a ninth for noise."""
    w = W.draw_workload(6, n, 1, v, param=param, with_sh=False)
    graphs = [_bwd_graph(w)]
    try:
        P.set_tuning(1, 1, v, 0, 4, 2 if v <= 8 else 4, 64 if 4 * n <= 32768 else 128)
        graphs.append(_bwd_graph(w))
    finally:
        P.set_tuning(1, 1, v, 0, 0, 0)
    built_in, four = _device_us(*graphs)
    assert built_in <= 1.11 * four, (built_in, four)


@pytest.mark.parametrize("n,k,v,param", [(16384, 1, 7, "quat"), (16385, 1, 7, "quat"), (40961, 1, 16, "quat"),
                                         (57344, 1, 16, "angles"), (57345, 1, 16, "angles"),
                                         (98305, 5, 8, "quat")])
def test_batch_follows_the_one_lobe_lines(n, k, v, param):
    test_batch_follows_the_shape_by_n(n, k, v, param)


def test_one_view_of_sg_waits_for_its_records_once():
    """A backward of 16 SG lobes on one lane against ASG's, which loads the same
    records and does more with them (0.81 of its time with the weights' loads
    ahead of the frame, 1.03 behind it); the bar lies between."""
    us = _device_us(*[_bwd_graph(W.draw_workload(7, 30000, 16, 1, family=family, with_sh=False))
                      for family in ("sg", "asg")])
    assert us[0] <= 0.94 * us[1], us


def test_batch_keeps_cheap_tiles_whole():
    """A plan's own tile size does not cut one-view, one-lobe scenes into tiles
    that cost less than their turn in the queue."""
    scenes = []
    for _ in range(16):
        d = upload(W.draw_workload(9, 8000, 1, 1, with_sh=False))
        d["grads"] = P.nasg_grad_buffers(1, 8000, "cuda")
        scenes.append(d)
    whole = P.NasgBatchPlan(scenes, tile_iters=8).n_items
    n_items = P.NasgBatchPlan(scenes).n_items
    assert whole < n_items and 16 * 8000 >= 384 * n_items


@pytest.mark.parametrize("n", [393216, 393217])
@pytest.mark.parametrize("v", [1, 2])
def test_sh_block_line(n, v):
    test_sh_shapes(n, v)
