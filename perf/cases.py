"""Timed workloads of the rasterizer framework, from its smallest calls to its largest.

Every case goes through the public entry points (`paper_2510_01767_amd.raster`) the way a block's
trainer, the camera selection, the partition or the densification calls them.  The scenes have the
shapes of `paper_2510_01767_amd.scenes` (unit cube, city block, city, cloud over a block), drawn on
the GPU from the seed.

  listed()             the cases
  draw(rng)            one more case of the same ranges
  prepare(case, seed)  what the program has in hand before the call
  run(state)           one pass; returns its outputs
  work(case)           bytes and operations one pass cannot do without
  exact(case, seed)    the outputs in float64 by plain torch, where that is affordable
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

PARAMS = ("means", "log_scales", "quats", "opacity_logits", "sh")
TILE = 16
# the images' sizes of the uneven batch: views cycle through them
UNEVEN = ((1920, 1080), (1600, 900), (960, 540), (1920, 1080), (1600, 900), (1920, 1080), (1600, 900), (960, 540))
LR = (1.6e-4, 5e-3, 1e-3, 5e-2, 2.5e-3, 1.25e-4)  # vanilla 3DGS learning rates


def listed():
    step = dict(kind="step", tile_w=16, tile_h=16, table=0, stats=True)
    return [
        # the smallest program: 2 000 flat-coloured Gaussians, one 128 x 128 view, a loss through autograd
        dict(step, name="tiny_autograd", form="autograd", scene="unit", n=2000, sh=0, views=1, width=128, height=128,
             batch=128, grid=4),
        # three small views of ragged sizes, replayed as one graph: launches and latency
        dict(step, name="ragged_graph", form="graph", scene="unit", n=3000, sh=3, views=3, width=150, height=97,
             batch=128, grid=4),
        # a trainer that takes one full-HD view at a time and brings its own image loss
        dict(kind="render", name="view_1080p", form="render", scene="block", n=1_000_000, sh=3, views=1, width=1920,
             height=1080, batch=128, grid=4, tile_w=16, tile_h=16, table=0, stats=True),
        # the default (plain) form: one launch chain per view, as a Rasterizer without options runs
        dict(step, name="plain_4views", form="plain", scene="block", n=1_500_000, sh=2, views=4, width=1600,
             height=900, batch=128, grid=4),
        # the batched step of a block: 3 M Gaussians, 16 views of uneven sizes, one graph
        dict(step, name="block_16views", form="graph", scene="block", n=3_000_000, sh=3, views=16, width=0, height=0,
             batch=256, grid=8),
        # a large block: 8 M Gaussians, 32 full-HD aerial views, launched eagerly
        dict(step, name="city_32views", form="eager", scene="city", n=8_000_000, sh=3, views=32, width=1920,
             height=1080, batch=256, grid=8, table=1),
        # depth-complexity stress: a low-opacity cloud over a block at 3840 x 2160
        dict(step, name="cloud_2160p", form="eager", scene="cloud", n=20_000_000, sh=3, views=8, width=3840,
             height=2160, batch=256, grid=8, table=1),
        # camera selection on a coarse model: depth renders, back-projection, coverage of 36 blocks
        dict(kind="depth", name="camera_select", scene="block", n=1_000_000, sh=3, views=8, width=1600, height=900,
             blocks=36, batch=256, grid=8, tile_w=16, tile_h=16, table=0),
        # the load-balanced partition of a scene into blocks, pixels resident on the GPU
        dict(kind="partition", name="partition", n=1_000_000, views=64, pixels=480 * 270, blocks=20, steps=3),
        # the optimizer step of a block
        dict(kind="adam", name="adam_dense", n=3_000_000, sh=3, visible_only=False),
        # selective densification and pruning with optimizer moments
        dict(kind="densify", name="densify", n=3_000_000, sh=3, selective=True, moments=True),
        # visibility cropping of a scene against a block's cameras
        dict(kind="visibility", name="visibility", scene="city", n=8_000_000, views=32, width=1920, height=1080),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step"] * 5 + ["render"] * 2 + ["depth", "adam", "densify", "visibility", "partition"])
    tile = rng.choice([(16, 16)] * 3 + [(32, 8), (8, 32)])
    c = dict(kind=kind, sh=rng.choice([0, 1, 2, 3, 3]), tile_w=tile[0], tile_h=tile[1],
             batch=rng.choice([64, 128, 256]), grid=rng.choice([4, 8]), table=rng.choice([0, 0, 1]))
    if kind in ("step", "render"):
        scene = rng.choice(["unit", "unit", "block", "block", "city", "cloud"])
        lo, hi, wmax = {"unit": (500, 20_000, 400), "block": (100_000, 4_000_000, 1920),
                        "city": (1_000_000, 8_000_000, 1920), "cloud": (500_000, 6_000_000, 2560)}[scene]
        n = _log(rng, lo, hi)
        views = rng.randint(1, 4) if scene in ("unit", "cloud") or kind == "render" else _log(rng, 1, 16)
        w = rng.randint(33, wmax) if scene == "unit" else rng.randint(wmax // 4, wmax)
        h = max(17, int(w * rng.uniform(0.5, 1.0)))
        form = "render" if kind == "render" else rng.choice(["autograd", "graph", "graph", "eager", "plain"])
        return dict(c, form=form, scene=scene, n=n, views=views, width=w, height=h, stats=rng.random() < 0.8)
    if kind == "depth":
        w = rng.randint(200, 1920)
        return dict(c, scene="block", n=_log(rng, 50_000, 2_000_000), views=rng.randint(1, 12), width=w,
                    height=int(w * 0.5625) + 1, blocks=rng.randint(1, 64))
    if kind == "partition":
        return dict(kind=kind, n=_log(rng, 20_000, 2_000_000), views=rng.randint(8, 96),
                    pixels=_log(rng, 4_000, 300_000), blocks=rng.randint(2, 36), steps=rng.choice([1, 2, 3, 3]))
    if kind == "adam":
        return dict(kind=kind, n=_log(rng, 1_000, 6_000_000), sh=c["sh"], visible_only=rng.random() < 0.5)
    if kind == "densify":
        return dict(kind=kind, n=_log(rng, 1_000, 4_000_000), sh=c["sh"], selective=rng.random() < 0.7,
                    moments=rng.random() < 0.8)
    return dict(kind=kind, scene=rng.choice(["block", "city"]), n=_log(rng, 10_000, 8_000_000),
                views=rng.randint(1, 32), width=rng.randint(300, 1920), height=rng.randint(200, 1080))


# ------------------------------------------------------------------ inputs


def _gen(seed, stream):
    return torch.Generator(device="cuda").manual_seed(1000003 * int(seed) + stream)


def _uniform(g, lo, hi, *size):
    return torch.rand(*size, generator=g, device="cuda") * (hi - lo) + lo


def _normal(g, mean, sd, *size):
    return torch.randn(*size, generator=g, device="cuda") * sd + mean


def _city_points(g, n, half, n_boxes):
    """60 % on the ground plane, 40 % on the walls and roofs of boxes, area weighted."""
    ng = round(0.6 * n)
    nb = n - ng
    ground = torch.cat([_uniform(g, -half, half, 2, ng), _normal(g, 0.0, 0.05, 1, ng)])
    centre = _uniform(g, -(half - 10.0), half - 10.0, 2, n_boxes)
    hx, hy = _uniform(g, 2.0, 10.0, n_boxes), _uniform(g, 2.0, 10.0, n_boxes)
    hz = _uniform(g, 5.0, 40.0, n_boxes)
    area = torch.stack([2 * hy * hz, 2 * hy * hz, 2 * hx * hz, 2 * hx * hz, 4 * hx * hy], 1).reshape(-1)
    edge = torch.cumsum(area.double(), 0)
    pick = torch.searchsorted(edge, torch.rand(nb, generator=g, device="cuda").double() * edge[-1])
    pick = pick.clamp(max=edge.numel() - 1)
    b, face = pick // 5, pick % 5
    u, v, w = _uniform(g, -1.0, 1.0, nb), _uniform(g, 0.0, 1.0, nb), _uniform(g, -1.0, 1.0, nb)
    one = torch.ones_like(u)
    x = torch.where(face == 0, one, torch.where(face == 1, -one, u))
    y = torch.where(face == 2, one, torch.where(face == 3, -one, torch.where(face == 4, w, u)))
    z = torch.where(face == 4, one, v)
    box = torch.stack([centre[0][b] + x * hx[b], centre[1][b] + y * hy[b], z * hz[b]])
    return torch.cat([ground, box], 1)


def _morton(means):
    """The order in which a trainer keeps its Gaussians: 10 bits an axis, interleaved."""
    lo = means.amin(1, keepdim=True)
    span = (means.amax(1, keepdim=True) - lo).clamp(min=1e-30)
    q = ((means - lo) / span * 1024.0).clamp(max=1023.0).to(torch.int64)
    code = torch.zeros(means.shape[1], dtype=torch.int64, device=means.device)
    for bit in range(10):
        for a in range(3):
            code |= ((q[a] >> bit) & 1) << (3 * bit + a)
    return torch.argsort(code)


def _gaussians(case, seed):
    """The parameters in storage order, float32 planes, and the block's half extent."""
    n, sh, scene = case["n"], case.get("sh", 3), case["scene"]
    g = _gen(seed, 1)
    half = {"unit": 1.0, "block": 100.0, "city": 500.0, "cloud": 100.0}[scene]
    logit_mu = torch.zeros(n, device="cuda")
    if scene == "unit":
        means = _uniform(g, -1.0, 1.0, 3, n)
    elif scene == "cloud":
        nc = n // 2
        means = torch.cat([_normal(g, 0.0, 20.0, 3, nc).clamp(-60.0, 60.0), _city_points(g, n - nc, 100.0, 200)], 1)
        logit_mu[:nc] = -2.0
    else:
        means = _city_points(g, n, half, 200 if scene == "block" else 2000)
    order = _morton(means) if scene != "unit" else torch.arange(n, device="cuda")
    means, logit_mu = means[:, order].contiguous(), logit_mu[order]
    K = (sh + 1) ** 2
    coef = _normal(g, 0.0, 0.2, 3 * K, n)
    coef[:3] = (_uniform(g, 0.0, 1.0, 3, n) - 0.5) / 0.28209479177387814
    quats = torch.nn.functional.normalize(_normal(g, 0.0, 1.0, 4, n), dim=0)
    return dict(means=means, log_scales=_normal(g, -3.0, 0.5, 3, n), quats=quats,
                opacity_logits=logit_mu + _normal(g, 0.0, 1.0, n), sh=coef), half


def _sizes(case):
    if case["width"]:
        w, h = case["width"], case["height"]
        ragged = case["scene"] == "unit" and case["views"] > 1  # small batches mix sizes
        return [(max(9, w >> k), max(9, h >> k)) if ragged else (w, h) for k in range(case["views"])]
    return [UNEVEN[k % len(UNEVEN)] for k in range(case["views"])]


def _cameras(case, seed, means):
    """Poses as the scene's captures have them; block views see 5 to 40 % of the Gaussians."""
    from paper_2510_01767_amd import scenes
    rng = random.Random(7919 * int(seed) + 5)
    scene, sizes = case["scene"], _sizes(case)
    some = means[:, :: max(1, means.shape[1] // 20000)].cpu().numpy()
    cams = []
    for k, (W, H) in enumerate(sizes):
        fx = 1500.0 * W / 1920.0
        if scene == "unit":
            a = 0.6 * k + rng.uniform(-0.1, 0.1)
            cams.append(scenes.look_at((4 * math.sin(a), -1.2 * math.cos(a), -4 * math.cos(a)), (0, 0, 0), W, H,
                                       float(min(W, H))))
            continue
        if scene == "cloud":
            a = 2 * math.pi * k / len(sizes) + rng.uniform(-0.1, 0.1)
            cams.append(scenes.look_at((112 * math.cos(a), 112 * math.sin(a), 84.0), (0, 0, 0), W, H, fx))
            continue
        for _ in range(60):
            if scene == "block":
                head, tgt = 2 * math.pi * k / len(sizes) + rng.uniform(-0.2, 0.2), (rng.gauss(0, 20), rng.gauss(0, 20))
                alt = rng.uniform(30.0, 150.0)
            else:
                head, tgt = rng.uniform(0, 2 * math.pi), (rng.uniform(-400, 400), rng.uniform(-400, 400))
                alt = rng.uniform(100.0, 300.0)
            cam = scenes.aerial_camera(tgt, head, rng.uniform(30.0, 60.0), alt, W, H, fx)
            if scene != "block" or 0.05 <= scenes.centre_in_view_fraction(cam, some) <= 0.40:
                break
        cams.append(cam)
    return cams


def _rasterizer(case, sizes, **more):
    from paper_2510_01767_amd.raster import Rasterizer
    mode = "plain" if case.get("form") == "plain" else "batched"
    return Rasterizer(case["n"], case.get("sh", 3), sizes, mode=mode, tile=(case["tile_w"], case["tile_h"]),
                      lds_batch=case["batch"], grid_per_cu=case["grid"], project_table=case["table"], **more)


def _views(case, seed):
    """Parameters, camera list, packed targets (also used as image gradients) of a case with views."""
    params, half = _gaussians(case, seed)
    cams = _cameras(case, seed, params["means"])
    pixels = sum(c["W"] * c["H"] for c in cams)
    return params, half, cams, _uniform(_gen(seed, 2), 0.0, 1.0, 3 * pixels)


def _blocks(case, seed, half):
    """A grid of blocks over the scene, a little jittered."""
    m = case["blocks"]
    side = math.ceil(math.sqrt(m))
    rng = random.Random(31 * int(seed) + 3)
    w, rows = 2 * half / side, []
    for k in range(m):
        x, y = -half + (k % side) * w + rng.uniform(-0.1, 0.1) * w, -half + (k // side) * w + rng.uniform(-0.1, 0.1) * w
        rows.append([x, y, -1.0, x + w, y + w, 60.0])
    return torch.tensor(rows, dtype=torch.float32, device="cuda")


def _planes(case, g, scale):
    n, K3 = case["n"], 3 * (case["sh"] + 1) ** 2
    shape = dict(means=(3, n), log_scales=(3, n), quats=(4, n), opacity_logits=(n,), sh=(K3, n))
    return {k: _normal(g, 0.0, scale, *shape[k]) for k in PARAMS}


def _adam_inputs(case, seed):
    """Parameters seen by a few small views (the optimizer's work does not depend on the views)."""
    view = dict(case, scene="block", views=2, width=320, height=180)
    params, _ = _gaussians(view, seed)
    cams = _cameras(view, seed, params["means"])
    g = _gen(seed, 3)
    grads, m, v = (_planes(case, g, 1e-4) for _ in range(3))
    return params, cams, grads, m, {k: x * x for k, x in v.items()}


def _densify_inputs(case, seed):
    """Which Gaussians densify or are pruned is drawn, how many is not: a tenth is over the gradient threshold
    (some of them split, the others cloned), as many outside the block are, and a twenty-fifth is transparent."""
    params, _ = _gaussians(dict(case, scene="block"), seed)
    g, n = _gen(seed, 4), case["n"]
    mixed = torch.randperm(n, generator=g, device="cuda")
    hot, out, low = mixed[:n // 10], mixed[n // 10:n // 5], mixed[n // 5:n // 5 + n // 25]
    inb = (torch.rand(n, generator=g, device="cuda") < 0.6).to(torch.uint8)
    inb[hot], inb[out] = 1, 0
    count = torch.randint(0, 12, (n,), generator=g, device="cuda", dtype=torch.int32)
    count[hot] += 1
    mean = torch.exp(_normal(g, -9.0, 0.8, n)).clamp(max=3.0e-4)
    mean[hot] = _uniform(g, 4.0e-4, 2.0e-3, hot.numel())
    if case["selective"]:
        mean[out] = _uniform(g, 4.0e-4, 2.0e-3, out.numel())
    params["opacity_logits"].clamp_(min=-1.7)
    params["opacity_logits"][low] = _uniform(g, -6.0, -2.0, low.numel())
    params["log_scales"].clamp_(max=-1.5)
    samples = _normal(g, 0.0, 1.0, 2, 3, n)
    m, v = (_planes(case, g, 1e-3), _planes(case, g, 1e-3)) if case["moments"] else (None, None)
    return params, count * mean, count, samples, inb if case["selective"] else None, m, v


DENSIFY = dict(grad_threshold=3.4e-4, clone_max_scale=0.07, min_opacity=0.15, max_world_scale=0.25)


def _partition_inputs(case, seed):
    g = _gen(seed, 5)
    half, V, P = 100.0, case["views"], case["pixels"]
    centers = _city_points(g, case["n"], half, 200)
    rng = random.Random(17 * int(seed) + 11)
    hot = (rng.uniform(-80, -30), rng.uniform(-80, -30))
    points, offsets = [], [0]
    for _ in range(V):  # most cameras look near one corner, the rest anywhere
        near = rng.random() < 0.6
        c = [h + rng.gauss(0, 15) if near else rng.uniform(-80, 80) for h in hot]
        r, k = rng.uniform(15, 45), rng.randint(P // 2, P)
        xy = [_uniform(g, a - r, a + r, k) for a in c]
        points.append(torch.stack([*xy, _uniform(g, 0.0, 1.0, k) ** 4 * 40.0]))
        offsets.append(offsets[-1] + k)
    host = centers.cpu().numpy()
    top = np.nextafter(np.float32(host[2].max()), np.float32(np.inf))
    aabb = np.array([-half, -half, host[2].min(), half, half, top], np.float32)
    return aabb, np.ascontiguousarray(host), torch.cat(points, 1).contiguous(), np.asarray(offsets, np.int64)


def prepare(case, seed):
    from paper_2510_01767_amd import raster
    kind, s = case["kind"], dict(case=case)
    if kind in ("step", "render", "depth"):
        params, half, cams, images = _views(case, seed)
        r = _rasterizer(case, [(c["W"], c["H"]) for c in cams])
        s.update(r=r, params=params, cams=raster.camera_tensor(cams), targets=images)
        if kind == "depth":
            s["blocks"] = _blocks(case, seed, half)
        elif kind == "render":
            s["targets"] = (images - 0.5) / images.numel()  # the gradient that the program's own loss gives
        if case.get("form") in ("autograd", "render"):
            s["leaves"] = {k: v.requires_grad_(True) for k, v in params.items()}
        if case.get("form") == "graph":
            s["stream"] = torch.cuda.Stream()
            s["stream"].wait_stream(torch.cuda.current_stream())
            with torch.cuda.stream(s["stream"]):
                r.capture(params, s["cams"], images, stats=case["stats"])
    elif kind == "visibility":
        params, half = _gaussians(case, seed)
        cams = _cameras(case, seed, params["means"])
        r = raster.Rasterizer(case["n"], 3, [(c["W"], c["H"]) for c in cams], mode="batched", capacity=1 << 20)
        s.update(r=r, params=params, cams=raster.camera_tensor(cams),
                 aabb=[-0.6 * half, -0.6 * half, -1.0, 0.6 * half, 0.6 * half, 50.0])
    elif kind == "adam":
        params, cams, grads, m, v = _adam_inputs(case, seed)
        r = raster.Rasterizer(case["n"], case["sh"], [(c["W"], c["H"]) for c in cams], mode="batched")
        if case["visible_only"]:
            r.forward(params, raster.camera_tensor(cams))
        s.update(r=r, params=params, grads=grads, m=m, v=v, t=0)
    elif kind == "densify":
        s["in"] = _densify_inputs(case, seed)
    else:
        s["in"] = _partition_inputs(case, seed)
    return s


# -------------------------------------------------------------------- run


def _step_outputs(r, loss, images, stats):
    out = dict(loss=loss, images=images, grads=[r.grads[k] for k in PARAMS])
    if stats:
        out.update(S=r.S, count=r.count)
    return out


def run(s):
    from paper_2510_01767_amd import raster
    case, kind = s["case"], s["case"]["kind"]
    if kind == "step":
        r, form = s["r"], case["form"]
        if form == "autograd":
            for p in s["leaves"].values():
                p.grad = None
            loss, images = raster.render_l1(s["leaves"], r, s["cams"], s["targets"])
            loss.backward()
            return dict(loss=loss.detach(), images=images, grads=[s["leaves"][k].grad for k in PARAMS])
        if form == "graph":
            # the statistics cover this step
            with torch.cuda.stream(s["stream"]):
                if case["stats"]:
                    r.S.zero_()
                    r.count.zero_()
                r.launch()
            torch.cuda.current_stream().wait_stream(s["stream"])
            return _step_outputs(r, r.loss, r.images, case["stats"])
        if case["stats"]:
            r.S.zero_()
            r.count.zero_()
        loss, images = r.step_l1(s["params"], s["cams"], s["targets"], stats=case["stats"])
        return _step_outputs(r, loss, images, case["stats"])
    if kind == "render":
        for p in s["leaves"].values():
            p.grad = None
        images = raster.render(s["leaves"], s["r"], s["cams"])
        images.backward(s["targets"])
        return dict(images=images.detach(), grads=[s["leaves"][k].grad for k in PARAMS])
    if kind == "depth":
        r = s["r"]
        images, depth = r.render_depth(s["params"], s["cams"])
        points = r.back_project(s["cams"], depth)
        counts, ratio, selected = r.camera_coverage(s["cams"], depth, s["blocks"], tau=0.1)
        return dict(images=images, depth=depth, points=points, counts=counts, ratio=ratio, selected=selected)
    if kind == "visibility":
        bits, keep, inb = s["r"].visibility_mask(s["params"], s["cams"], aabb=s["aabb"])
        return dict(bits=bits, keep=keep, in_block=inb)
    if kind == "adam":
        s["t"] += 1
        s["r"].adam_step(s["params"], s["grads"], s["m"], s["v"], LR, s["t"], visible_only=case["visible_only"])
        return dict(params=s["params"], m=s["m"], v=s["v"])
    if kind == "densify":
        params, S, count, samples, inb, m, v = s["in"]
        out, mo, vo, parent = raster.densify(params, S, count, samples, in_block=inb, m=m, v=v, **DENSIFY)
        return dict(params=out, m=mo, v=vo, parent=parent)
    aabb, centers, points, offsets = s["in"]
    blocks, assign, workload = raster.partition_blocks_device(aabb, centers, points, offsets, case["blocks"],
                                                              refine_steps=case["steps"])
    return dict(blocks=blocks, assign=assign, workload=workload)


# ------------------------------------------------------------------- work

# entries blended into a pixel of each scene, and flops of one blended pair forward and in both directions
BLENDED = {"unit": 20, "block": 19, "city": 15, "cloud": 100}
FLOPS_FWD, FLOPS_BOTH = 25, 79


def work(case):
    """Inputs read once, outputs written once; the blended pairs' arithmetic."""
    n, kind = case["n"], case["kind"]
    planes = 11 + 3 * (case.get("sh", 3) + 1) ** 2
    if kind == "adam":
        return dict(bytes=28 * planes * n, flops=12 * planes * n)
    if kind == "densify":
        return dict(bytes=(3 if case["moments"] else 1) * 8 * planes * n + 40 * n, flops=10 * n)
    if kind == "partition":
        total = 0.75 * case["views"] * case["pixels"]
        return dict(bytes=12 * total + 12 * n, flops=6 * total * case["blocks"])
    if kind == "visibility":
        return dict(bytes=(44 + 6) * n, flops=30 * n * case["views"])
    P = sum(w * h for w, h in _sizes(case))
    pairs = P * BLENDED[case["scene"]]
    if kind == "depth":
        return dict(bytes=4 * planes * n + 40 * P, flops=FLOPS_FWD * pairs)
    extra = 24 * P + (8 * n if case["stats"] else 0)
    return dict(bytes=8 * planes * n + extra, flops=FLOPS_BOTH * pairs)


# ------------------------------------------------------- the same in float64


def _basis(D, d):
    """Real orthonormal spherical harmonics with the Condon-Shortley phase at unit vectors d [m][3]."""
    x, y, z = d.unbind(1)
    c = lambda a, b: math.sqrt(a / (b * math.pi))
    out = [torch.full_like(x, c(1, 4))]
    if D > 0:
        out += [-c(3, 4) * y, c(3, 4) * z, -c(3, 4) * x]
    if D > 1:
        out += [c(15, 4) * x * y, -c(15, 4) * y * z, c(5, 16) * (3 * z * z - 1), -c(15, 4) * x * z,
                c(15, 16) * (x * x - y * y)]
    if D > 2:
        out += [-c(35, 32) * y * (3 * x * x - y * y), c(105, 4) * x * y * z, -c(21, 32) * y * (5 * z * z - 1),
                c(7, 16) * z * (5 * z * z - 3), -c(21, 32) * x * (5 * z * z - 1), c(105, 16) * z * (x * x - y * y),
                -c(35, 32) * x * (x * x - 3 * y * y)]
    return torch.stack(out, 1)


def _project(p, sh, cam, tile):
    """Every Gaussian of p (float64 leaves) in one view: what compositing reads, and who is visible."""
    f64 = lambda a: torch.as_tensor(np.asarray(a, np.float64), device="cuda")
    R, t = f64(cam["R"]), f64(cam["t"])
    fx, fy, cx, cy = (float(cam[k]) for k in ("fx", "fy", "cx", "cy"))
    W, H = cam["W"], cam["H"]
    mu = p["means"].T
    tc = mu @ R.T + t
    z = torch.where(tc[:, 2] > 0.01, tc[:, 2], torch.ones_like(tc[:, 2]))
    ux, uy = tc[:, 0] / z, tc[:, 1] / z
    mean = torch.stack([fx * ux + cx, fy * uy + cy], 1)
    lim = [float(np.float32(1.3)) * 0.5 * s / f for s, f in ((W, fx), (H, fy))]
    u, v = ux.clamp(-lim[0], lim[0]), uy.clamp(-lim[1], lim[1])
    zero = torch.zeros_like(z)
    J = torch.stack([fx / z, zero, -fx * u / z, zero, fy / z, -fy * v / z], 1).reshape(-1, 2, 3)
    w, x, y, k = (p["quats"] / p["quats"].norm(dim=0, keepdim=True)).unbind(0)
    rot = torch.stack([1 - 2 * (y * y + k * k), 2 * (x * y - w * k), 2 * (x * k + w * y), 2 * (x * y + w * k),
                       1 - 2 * (x * x + k * k), 2 * (y * k - w * x), 2 * (x * k - w * y), 2 * (y * k + w * x),
                       1 - 2 * (x * x + y * y)], 1).reshape(-1, 3, 3)
    L = (J @ R) @ (rot * torch.exp(p["log_scales"]).T[:, None, :])
    a = (L[:, 0] * L[:, 0]).sum(1) + float(np.float32(0.3))
    b = (L[:, 0] * L[:, 1]).sum(1)
    c = (L[:, 1] * L[:, 1]).sum(1) + float(np.float32(0.3))
    det = a * c - b * b
    conic = torch.stack([c, -b, a], 1) / det[:, None]
    eye = mu + R.T @ t
    Y = _basis(sh, eye / eye.norm(dim=1, keepdim=True))
    colour = torch.relu(torch.einsum("kcn,nk->nc", p["sh"].reshape(-1, 3, mu.shape[0]), Y) + 0.5)
    with torch.no_grad():
        r = torch.ceil(3.0 * torch.sqrt(0.5 * (a + c) + torch.sqrt((0.5 * (a - c)) ** 2 + b * b)))
        size = torch.tensor(tile, dtype=torch.float64, device="cuda")
        grid = torch.tensor([(W + tile[0] - 1) // tile[0], (H + tile[1] - 1) // tile[1]], device="cuda")
        lo = torch.floor((mean - r[:, None]) / size)
        hi = torch.floor((mean + r[:, None]) / size)
        vis = (tc[:, 2] > float(np.float32(0.01))) & (tc[:, 2] < 1e10) & (det > 0)
        vis &= ((hi >= 0) & (lo <= grid - 1)).all(1)
        rect = (lo.clamp(min=0).to(torch.int64), torch.minimum(hi, (grid - 1).double()).to(torch.int64))
    return mean, conic, torch.sigmoid(p["opacity_logits"]), colour, tc[:, 2], vis, rect, grid


def _visible(p, sh, cam, tile):
    """Indices of the Gaussians visible in a view, found in slices."""
    n, got = p["means"].shape[1], []
    with torch.no_grad():
        for a in range(0, n, 1 << 20):
            part = {k: v[..., a:a + (1 << 20)].double() for k, v in p.items()}
            part["sh"] = part["sh"][:3]
            got.append(_project(part, 0, cam, tile)[5].nonzero()[:, 0] + a)
    return torch.cat(got)


def _composite(rec, depth, lists, origin, W, H, tile, target, scale, gradient):
    """One group of tiles: lists [t][L] of record numbers (-1 past a list's end), origin [t][2].  Adds the
    records' gradients; returns (x, y, colour, depth) of the pixels inside the view."""
    mean, conic, opac, colour = rec
    valid = lists >= 0
    idx = lists.clamp(min=0)
    k = torch.arange(tile[0] * tile[1], device="cuda")
    x, y = origin[:, :1] + k % tile[0], origin[:, 1:] + k // tile[0]
    m, q = mean[idx], conic[idx]
    dx, dy = (x + 0.5)[:, None, :] - m[..., 0:1], (y + 0.5)[:, None, :] - m[..., 1:2]
    power = -0.5 * (q[..., 0:1] * dx * dx + q[..., 2:3] * dy * dy) - q[..., 1:2] * dx * dy
    alpha = torch.clamp(opac[idx][..., None] * torch.exp(power.clamp(max=0.0)), max=float(np.float32(0.99)))
    hit = valid[..., None] & (alpha >= float(np.float32(1.0 / 255.0))) & (power <= 0)
    alpha = torch.where(hit, alpha, torch.zeros_like(alpha))
    logt = torch.cumsum(torch.log1p(-alpha), 1)
    with torch.no_grad():
        alive = torch.exp(logt) >= float(np.float32(1e-4))
    weight = alpha * torch.exp(logt - torch.log1p(-alpha)) * alive
    inside = (x < W) & (y < H)
    out = torch.einsum("tlp,tlc->tcp", weight, colour[idx])
    with torch.no_grad():
        far = (weight * depth[idx][..., None]).sum(1)
    if target is not None:
        want = target[:, y.clamp(max=H - 1), x.clamp(max=W - 1)].transpose(0, 1)
        g = want if gradient else torch.sign(out.detach() - want) * scale
        out.backward(torch.where(inside[:, None, :], g, torch.zeros_like(g)))
    o = out.detach().transpose(0, 1)[:, inside]
    return x[inside], y[inside], o, far[inside]


def _exact_views(case, seed):
    params, half, cams, images = _views(case, seed)
    tile, sh, n = (case["tile_w"], case["tile_h"]), case["sh"], case["n"]
    kind = case["kind"]
    backward = kind != "depth"
    grads = {k: torch.zeros_like(v, dtype=torch.float64) for k, v in params.items()}
    S, count = torch.zeros(n, dtype=torch.float64, device="cuda"), torch.zeros(n, dtype=torch.int32, device="cuda")
    loss, all_images, all_depth, at = 0.0, [], [], 0
    for cam in cams:
        W, H = cam["W"], cam["H"]
        target = images[at:at + 3 * W * H].reshape(3, H, W).double()
        if kind == "render":
            target = ((images[at:at + 3 * W * H] - 0.5) / images.numel()).reshape(3, H, W).double()
        at += 3 * W * H
        scale = 1.0 / (3.0 * W * H * len(cams))
        sel = _visible(params, sh, cam, tile)
        leaf = {k: v.detach()[..., sel].double().requires_grad_(backward) for k, v in params.items()}
        mean, conic, opac, colour, depth, _, (lo, hi), grid = _project(leaf, sh, cam, tile)
        rec = [v.detach().requires_grad_(backward) for v in (mean, conic, opac, colour)]
        depth = depth.detach()
        wide = hi[:, 0] - lo[:, 0] + 1
        many = wide * (hi[:, 1] - lo[:, 1] + 1)
        who = torch.repeat_interleave(torch.arange(sel.numel(), device="cuda"), many)
        j = torch.arange(who.numel(), device="cuda") - torch.repeat_interleave(many.cumsum(0) - many, many)
        tid = (lo[who, 1] + j // wide[who]) * grid[0] + lo[who, 0] + j % wide[who]
        # front to back: by tile, then the float32 depth, then the index
        order = torch.argsort((tid << 32) | depth.float().view(torch.int32).to(torch.int64)[who], stable=True)
        who, tid = who[order], tid[order]
        tiles = int(grid[0] * grid[1])
        length = torch.bincount(tid, minlength=tiles)
        start = length.cumsum(0) - length
        image = torch.zeros(3, H, W, dtype=torch.float64, device="cuda")
        far = torch.zeros(H, W, dtype=torch.float64, device="cuda")
        by_length = torch.argsort(length, descending=True)
        lengths, a = length[by_length].tolist(), 0
        while a < tiles:
            L = max(1, lengths[a])
            t = by_length[a:a + max(1, 40_000_000 // (L * tile[0] * tile[1]))]
            a += t.numel()
            col = torch.arange(L, device="cuda")
            have = col < length[t][:, None]
            lists = torch.full(have.shape, -1, dtype=torch.int64, device="cuda")
            if who.numel():
                lists = torch.where(have, who[(start[t][:, None] + col).clamp(max=who.numel() - 1)], lists)
            if not sel.numel():
                continue
            origin = torch.stack([t % grid[0] * tile[0], t // grid[0] * tile[1]], 1)
            x, y, o, d = _composite(rec, depth, lists, origin, W, H, tile, target if backward else None, scale,
                                    kind == "render")
            image[:, y, x], far[y, x] = o, d
        loss += float((image - target).abs().sum()) * scale
        all_images.append(image.reshape(-1))
        all_depth.append(far.reshape(-1))
        if backward and sel.numel() and rec[0].grad is not None:
            torch.autograd.backward([mean, conic, opac, colour], [v.grad for v in rec])
            for k in PARAMS:
                grads[k][..., sel] += leaf[k].grad
            S[sel] += len(cams) * rec[0].grad.norm(dim=1)
            count[sel] += 1
    flat = torch.cat(all_images)
    if kind == "depth":
        points, depth = [], torch.cat(all_depth)
        for cam, d in zip(cams, all_depth):
            R, t = (torch.as_tensor(np.asarray(cam[k], np.float64), device="cuda") for k in ("R", "t"))
            k = torch.arange(d.numel(), device="cuda")
            u = (k % cam["W"] + 0.5 - float(cam["cx"])) / float(cam["fx"])
            v = (torch.div(k, cam["W"], rounding_mode="floor") + 0.5 - float(cam["cy"])) / float(cam["fy"])
            points.append(R.T @ (torch.stack([d * u, d * v, d]) - t[:, None]))
        return dict(images=flat, depth=depth, points=torch.cat(points, 1), counts=None, ratio=None, selected=None)
    g = [grads[k] for k in PARAMS]
    if kind == "render":
        return dict(images=flat, grads=g)
    if case["form"] == "autograd":
        return dict(loss=torch.tensor(loss, dtype=torch.float64), images=flat, grads=g)
    out = dict(loss=torch.tensor([loss], dtype=torch.float64), images=flat, grads=g)
    if case["stats"]:
        out.update(S=S, count=None)
    return out


def _exact_adam(case, seed):
    params, cams, grads, m, v = _adam_inputs(case, seed)
    b1, b2, eps = (float(np.float32(a)) for a in (0.9, 0.999, 1e-15))
    seen = torch.ones(case["n"], dtype=torch.bool, device="cuda")
    if case["visible_only"]:
        seen.zero_()
        for cam in cams:
            seen[_visible(params, case["sh"], cam, (TILE, TILE))] = True
    out = dict(params={}, m={}, v={})
    for k, name in enumerate(PARAMS):
        lr = torch.full((params[name].shape[0],), LR[min(k, 4)], dtype=torch.float64, device="cuda")
        if name == "sh":
            lr[3:] = LR[5]
        lr = (lr.float().double()[:, None] if params[name].dim() == 2 else float(np.float32(LR[k])))
        p, g, m0, v0 = (d[name].double() for d in (params, grads, m, v))
        m1, v1 = b1 * m0 + (1 - b1) * g, b2 * v0 + (1 - b2) * g * g
        p1 = p - lr / (1 - b1) * m1 / (torch.sqrt(v1) / math.sqrt(1 - b2) + eps)
        out["params"][name], out["m"][name], out["v"][name] = (torch.where(seen, x, y) for x, y in
                                                               ((p1, p), (m1, m0), (v1, v0)))
    return out


def _exact_densify(case, seed):
    params, S, count, samples, inb, m, v = _densify_inputs(case, seed)
    f = {k: float(np.float32(a)) for k, a in DENSIFY.items()}
    big = params["log_scales"].amax(0)
    opaque = params["opacity_logits"].double() >= math.log(f["min_opacity"] / (1 - f["min_opacity"]))
    hot = (count > 0) & (S.double() >= f["grad_threshold"] * count.double())
    if inb is not None:
        hot &= inb.bool()
    split = hot & (big.double() > math.log(f["clone_max_scale"]))
    shrink = float(np.float32(math.log(1.6)))
    top = torch.where(split, (big - shrink), big).double()
    keep = opaque & (top <= math.log(f["max_world_scale"]))
    parent = torch.repeat_interleave(torch.arange(case["n"], device="cuda"), torch.where(hot, 2, 1) * keep)
    second = torch.zeros_like(parent, dtype=torch.bool)
    second[1:] = parent[1:] == parent[:-1]
    is_split = split[parent]
    out = {k: params[k][..., parent].double() for k in PARAMS}
    w, x, y, z = torch.nn.functional.normalize(out["quats"], dim=0).unbind(0)
    s = torch.exp(out["log_scales"])
    d = s * torch.where(second, samples[1][:, parent], samples[0][:, parent]).double()
    rot = [[1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y)],
           [2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x)],
           [2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)]]
    move = torch.stack([r[0] * d[0] + r[1] * d[1] + r[2] * d[2] for r in rot])
    out["means"] = torch.where(is_split, out["means"] + move, out["means"])
    out["log_scales"] = torch.where(is_split, out["log_scales"] - math.log(1.6), out["log_scales"])
    fresh = is_split | second
    moment = lambda a: None if a is None else {k: torch.where(fresh, 0.0, a[k][..., parent].double()) for k in PARAMS}
    return dict(params=out, m=moment(m), v=moment(v), parent=None)


def exact(case, seed):
    kind = case["kind"]
    if kind in ("visibility", "partition"):  # whole numbers, and coordinates that are copies of inputs
        return None
    if kind == "adam":
        return _exact_adam(case, seed)
    if kind == "densify":
        return _exact_densify(case, seed)
    pairs = sum(w * h for w, h in _sizes(case)) * {"unit": 200, "block": 320, "city": 250, "cloud": 1200}[case["scene"]]
    if pairs * (0.4 if kind == "depth" else 1.0) > 1.8e10:
        return None
    return _exact_views(case, seed)
