"""The work that programs built on this package have it do, as cases that can
be timed and compared: stereo frames, single renders, batches, the learned
repair (inference and training), the reprojection with hole classification,
and the pair sort.

A case is a dict of plain values.  `listed()` gives the cases at the sizes of
the package's own workloads, `draw(rng)` more of the same ranges; `prepare`
makes what a program holds before the call, `run` makes one pass through the
public entry points, `work` says what a pass cannot do without, and `exact`
gives its results in 64 bits where that is quick.
"""
import math

import numpy as np
import torch

from paper_2609_30741_amd import api, batch, repair, synth

DEV = "cuda"
BASELINE = synth.BASELINE_IPD


def listed():
    return [
        # One render of a small cloud in a small ragged window: the smallest
        # call, where latency and the number of launches count.
        dict(name="mono_cube_129x65", kind="mono", scene="cube", n=1500, w=129, h=65, pose=0.1),
        # The 10k-surfel cube seen by both eyes at 256x256: a small frame.
        dict(name="stereo_cube_256", kind="stereo", scene="cube", n=10_000, w=256, h=256, pose=0.0, tile=16,
             margin=32, center_roi=1, edge_bounds=0, view_colour=0),
        # The object-centric frame: a 300k-surfel shell at 800x600 per eye.
        dict(name="stereo_sphere_800x600", kind="stereo", scene="sphere", n=300_000, w=800, h=600, pose=0.3, tile=16,
             margin=32, center_roi=1, edge_bounds=0, view_colour=0),
        # The unbounded 1M-surfel frame at 1600x1064 per eye, half way along
        # its path (the headline workload).
        dict(name="stereo_unbounded_1600x1064", kind="stereo", scene="unbounded", n=1_000_000, w=1600, h=1064,
             pose=0.5, tile=16, margin=32, center_roi=1, edge_bounds=0, view_colour=0),
        # The serving frame, 2064x2208 per eye, near the end of the path,
        # where the ROIs cover much of the image.
        dict(name="stereo_unbounded_2064x2208", kind="stereo", scene="unbounded", n=1_000_000, w=2064, h=2208,
             pose=0.9, tile=16, margin=32, center_roi=1, edge_bounds=0, view_colour=0),
        # One eye of the two-pass form on a large shell at 1920x1080.
        dict(name="mono_sphere_1920x1080", kind="mono", scene="sphere", n=1_200_000, w=1920, h=1080, pose=0.7),
        # Eight mixed pairs over four resident scenes, captured into a graph
        # and replayed: the batched form.
        dict(name="batch_8_pairs", kind="batch", pairs=8, scale=1.0),
        # The repair network over one 800x600 frame, with its error channel.
        dict(name="repair_800x600", kind="repair", batch=1, w=800, h=600),
        # The same over a serving frame.
        dict(name="repair_2064x2208", kind="repair", batch=1, w=2064, h=2208),
        # One training step on eight 128x128 crops, the trainer's default.
        dict(name="train_8x128x128", kind="train", batch=8, w=128, h=128),
        # Reprojection and hole classification of a given dominant image, a
        # ragged size and a toed-in rig (rows not preserved), per-edge bounds.
        dict(name="warp_1603x1061", kind="warp", w=1603, h=1061, toe=2.0, occluders=6, passes=2, edge_bounds=1),
        # The pair sort at the key count and tile bits of a 1600x1064 frame.
        dict(name="sort_19600000x13", kind="sort", n=19_600_000, bits=13),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["mono", "mono", "stereo", "stereo", "stereo", "batch", "repair", "train", "warp", "sort"])
    if kind in ("mono", "stereo"):
        c = dict(kind=kind, scene=rng.choice(["cube", "sphere", "unbounded"]), n=_log(rng, 1500, 1_000_000),
                 w=_log(rng, 96, 2064), h=_log(rng, 64, 2208), pose=round(rng.random(), 3))
        if kind == "stereo":
            c.update(tile=rng.choice([16, 16, 16, 8, 32]), margin=rng.choice([32, 32, 16, 0, 64]),
                     center_roi=int(rng.random() < 0.85), edge_bounds=int(rng.random() < 0.2),
                     view_colour=int(rng.random() < 0.15))
        return c
    if kind == "batch":
        return dict(kind=kind, pairs=rng.randint(2, 8), scale=round(rng.uniform(0.05, 1.0), 3))
    if kind == "repair":
        w, h = 4 * _log(rng, 16, 516), 4 * _log(rng, 16, 552)
        return dict(kind=kind, batch=rng.randint(1, 4) if w * h < 500_000 else 1, w=w, h=h)
    if kind == "train":
        return dict(kind=kind, batch=rng.randint(1, 12), w=4 * _log(rng, 8, 64), h=4 * _log(rng, 8, 64))
    if kind == "warp":
        return dict(kind=kind, w=_log(rng, 64, 2752), h=_log(rng, 64, 2208), toe=rng.choice([0.0, 0.0, 2.0, -1.0]),
                    occluders=rng.randint(2, 12), passes=rng.choice([2, 2, 1, 4]),
                    edge_bounds=int(rng.random() < 0.3))
    return dict(kind=kind, n=_log(rng, 1000, 19_600_000), bits=rng.randint(1, 32))


# --------------------------------------------------------------------------
# Inputs, made on the GPU from the seed: the scenes of the package's
# workloads (same distributions), images as the reprojection leaves them.
# --------------------------------------------------------------------------

def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _normal(g, *shape):
    return torch.randn(*shape, generator=g, device=DEV)


def _uniform(g, *shape):
    return torch.rand(*shape, generator=g, device=DEV)


def _dirs(g, n):
    d = _normal(g, 3, n)
    return d / d.norm(dim=0, keepdim=True)


def _scene(kind, n, seed):
    """A scene of n surfels of one of the package's three kinds."""
    g = _gen(seed)
    log_scale = -3.5 + 0.5 * _normal(g, 2, n)
    quat = _normal(g, 4, n)
    quat = quat / quat.norm(dim=0, keepdim=True)
    if kind == "cube":
        pos = 2.0 * _uniform(g, 3, n) - 1.0
        opacity = torch.sigmoid(1.5 * _normal(g, n))
        sh = (_uniform(g, 3, n) - 0.5) / 0.28209479177387814
        degree = 0
    else:
        degree = 3
        sh = 0.2 * _normal(g, 48, n)
        if kind == "sphere":
            d = _dirs(g, n)
            pos = d * (1.0 + 0.02 * _normal(g, n))
            opacity = torch.sigmoid(1.0 + _normal(g, n))
            # A spin about z, then the rotation that takes z to d.
            half = math.pi * _uniform(g, n)
            c, s = torch.cos(half), torch.sin(half)
            a = torch.stack([1.0 + d[2], -d[1], d[0]])
            a = a / a.norm(dim=0, keepdim=True).clamp_min(1e-12)
            quat = torch.stack([a[0] * c, a[1] * c + a[2] * s, a[2] * c - a[1] * s, a[0] * s])
            quat = quat / quat.norm(dim=0, keepdim=True)
        else:
            n_in = int(round(0.7 * n))
            r = torch.cat([_uniform(g, n_in) ** (1.0 / 3.0), torch.exp(math.log(20.0) * _uniform(g, n - n_in))])
            pos = _dirs(g, n) * r
            opacity = torch.sigmoid(2.0 * _normal(g, n))
    f = lambda t: t.float().cpu().numpy()  # noqa: E731
    return synth.Scene(n, degree, f(pos), f(quat), f(torch.exp(log_scale)), f(opacity), f(sh))


def _cameras(kind, w, h, pose):
    up = (0.0, 0.0, 1.0)
    th = 2.0 * math.pi * pose
    if kind == "cube":  # at distance 4
        cam = synth.look_at((4.0 * math.sin(th), -4.0 * math.cos(th), 0.0), (0.0, 0.0, 0.0), up, w, h, 300.0 * w / 256)
    elif kind == "sphere":  # an orbit of radius 3
        cam = synth.look_at((3.0 * math.cos(th), 3.0 * math.sin(th), 0.0), (0.0, 0.0, 0.0), up, w, h, 1.375 * w)
    else:  # a straight path into the scene
        y = -6.0 + 4.5 * pose
        cam = synth.look_at((0.0, y, 0.0), (0.0, y + 1.0, 0.0), up, w, h, 1300.0 * w / 1600)
    return cam, synth.affiliated(cam, BASELINE)


def _field(g, batch, channels, h, w, cell):
    """A smooth random field in [0, 1]."""
    grid = _uniform(g, batch, channels, h // cell + 2, w // cell + 2)
    return torch.nn.functional.interpolate(grid, size=(h, w), mode="bilinear", align_corners=True).contiguous()


def _warped(seed, b, h, w):
    """Images as the reprojection hands them to the repair network: smooth
    colours, about 6% holes (thin slits and a strip at one side), depth with
    an infinite background; and the target without holes."""
    g = _gen(seed)
    target = (0.8 * _field(g, b, 3, h, w, 24) + 0.2 * _field(g, b, 3, h, w, 5)).contiguous()
    z = 2.0 + 4.0 * _field(g, b, 1, h, w, 40)[:, 0]
    z = torch.where(_field(g, b, 1, h, w, 48)[:, 0] < 0.15, torch.full_like(z, math.inf), z)
    slit = _field(g, b, 1, h, w, 9)[:, 0]
    hole = ((slit > 0.49) & (slit < 0.505)) | (torch.arange(w, device=DEV) >= w - max(1, w // 40))
    rgb = torch.where(hole[:, None], torch.zeros_like(target), target + 0.01 * _normal(g, b, 3, h, w))
    z = torch.where(hole, torch.full_like(z, math.inf), z)
    return rgb.contiguous(), z.contiguous(), hole.to(torch.uint8).contiguous(), target


def _toed(cam, baseline, degrees):
    """The affiliated eye, turned towards the dominant one by some degrees."""
    c = synth.affiliated(cam, baseline)
    a = math.radians(degrees)
    turn = np.array([[math.cos(a), 0.0, -math.sin(a)], [0.0, 1.0, 0.0], [math.sin(a), 0.0, math.cos(a)]])
    if degrees:
        c.R = c.R @ turn
    return c


def _stage_images(seed, w, h, occluders):
    """A dominant image with its depth proxy: a sloped background, nearer
    rectangles and an empty blob."""
    g = _gen(seed)
    u = _uniform(g, 8 + 5 * occluders).tolist()
    yy, xx = torch.meshgrid(torch.arange(h, device=DEV) / h, torch.arange(w, device=DEV) / w, indexing="ij")
    z = (3.0 + 3.0 * u[0]) * (1.0 + 0.6 * (u[1] - 0.5) * (xx - 0.5) + 0.6 * (u[2] - 0.5) * (yy - 0.5))
    rgb = 0.2 + 0.6 * _field(g, 1, 3, h, w, 16)[0]
    for k in range(occluders):
        x0, y0, dx, dy, zf = u[8 + 5 * k:13 + 5 * k]
        m = (xx >= x0) & (xx <= x0 + 0.05 + 0.3 * dx) & (yy >= y0) & (yy <= y0 + 0.05 + 0.3 * dy)
        z = torch.where(m, torch.full_like(z, 0.6 + 1.4 * zf), z)
        rgb = torch.where(m, (0.5 * rgb + 0.5 * dx).clamp(0, 1), rgb)
    d2 = ((xx - u[3]) ** 2 + (yy - u[4]) ** 2) / (0.1 / math.pi)
    alpha = (1.5 * (d2 - 0.5)).clamp(0.0, 1.0) * (0.97 + 0.03 * _uniform(g, h, w))
    return (rgb * alpha).contiguous(), (z * alpha).contiguous(), alpha.contiguous()


def _stereo_out(cam, tile):
    h, w = cam.height, cam.width
    f = lambda *s: torch.zeros(s, device=DEV)  # noqa: E731
    return dict(rgb_dom=f(3, h, w), depth_raw_dom=f(h, w), alpha_dom=f(h, w), rgb_aff=f(3, h, w), z_aff=f(h, w),
                alpha_aff=f(h, w), cls_aff=torch.zeros((h, w), dtype=torch.uint8, device=DEV),
                labels=torch.zeros((h, w), dtype=torch.int32, device=DEV),
                boxes=torch.zeros((4096, 6), dtype=torch.int32, device=DEV),
                n_boxes=torch.zeros(1, dtype=torch.int32, device=DEV),
                tile_mask=torch.zeros(((h + tile - 1) // tile, (w + tile - 1) // tile), dtype=torch.uint8, device=DEV))


def _batch_pairs(case, seed):
    """Pair i on resident scene i mod 4 (cube and shell kinds in turn), each
    with a resolution, a pose and an ROI tile size and margin of its own."""
    rng = np.random.default_rng(seed + 100)
    kinds = ("cube", "sphere", "cube", "sphere")
    sizes = [max(1000, int(case["scale"] * n)) for n in (50_000, 200_000, 600_000, 1_200_000)]
    scenes = [api.DeviceScene(_scene(k, n, seed + i)) for i, (k, n) in enumerate(zip(kinds, sizes))]
    pairs = []
    for i in range(case["pairs"]):
        w, h = synth.BATCH_RESOLUTIONS[i * 3 % 4]
        cd, ca = _cameras(kinds[i % 4], w, h, float(rng.uniform()))
        roi = api.Roi(tile=(16, 8, 32)[i % 3], margin=(32, 16)[i % 2])
        pairs.append((scenes[i % 4], cd, ca, roi))
    return pairs


def prepare(case, seed):
    kind = case["kind"]
    if kind == "mono":
        cam, _ = _cameras(case["scene"], case["w"], case["h"], case["pose"])
        scene = api.DeviceScene(_scene(case["scene"], case["n"], seed))
        ctx = api.Context(sync=True)
        out = ctx.render_dominant(scene, cam)  # a synchronous frame sizes the workspace
        ctx.set_sync(False)
        return dict(kind=kind, ctx=ctx, scene=scene, cam=cam, out=out)
    if kind == "stereo":
        cd, ca = _cameras(case["scene"], case["w"], case["h"], case["pose"])
        scene = api.DeviceScene(_scene(case["scene"], case["n"], seed))
        roi = api.Roi(tile=case["tile"], margin=case["margin"], center_roi=bool(case["center_roi"]),
                      edge_bounds=case["edge_bounds"], view_colour=case["view_colour"])
        ctx = api.Context(sync=True)
        out = ctx.render_stereo(scene, cd, ca, roi=roi, out=_stereo_out(cd, case["tile"]))
        ctx.set_sync(False)
        return dict(kind=kind, ctx=ctx, scene=scene, cd=cd, ca=ca, roi=roi, out=out)
    if kind == "batch":
        stream = torch.cuda.Stream()
        with torch.cuda.stream(stream):
            ctx = api.Context(sync=False)
            b = batch.StereoBatch(ctx, _batch_pairs(case, seed))
            for o in b.outs:
                o["boxes"].zero_()
            b.capture()
        stream.synchronize()
        return dict(kind=kind, batch=b, stream=stream)
    if kind in ("repair", "train"):
        rgb, z, hole, target = _warped(seed, case["batch"], case["h"], case["w"])
        s = dict(kind=kind, net=repair.Repair(seed=seed), rgb=rgb, z=z, hole=hole, target=target)
        if kind == "repair":
            s.update(out=torch.zeros_like(rgb), err=torch.zeros_like(z))
        return s
    if kind == "warp":
        w, h = case["w"], case["h"]
        src = synth.look_at((0.0, -4.0, 0.0), (0.0, 0.0, 0.0), (0.0, 0.0, 1.0), w, h, 1.2 * w)
        dst = _toed(src, BASELINE, case["toe"])
        rgb, depth, alpha = _stage_images(seed, w, h, case["occluders"])
        o = _stereo_out(src, 16)
        warp = dict(rgb=o["rgb_aff"], z=o["z_aff"], alpha=o["alpha_aff"], hole=o["cls_aff"],
                    depth_range=torch.zeros(2, device=DEV))
        cls = {k: o[k] for k in ("labels", "boxes", "n_boxes", "tile_mask")}
        ctx = api.Context(sync=False)
        ctx.workspace(0, w, h, 0)
        return dict(kind=kind, ctx=ctx, src=src, dst=dst, rgb=rgb, depth=depth, alpha=alpha, warp=warp, cls=cls,
                    roi=api.Roi(gap_passes=case["passes"], edge_bounds=case["edge_bounds"]))
    g = _gen(seed)
    keys = torch.randint(0, 1 << case["bits"], (case["n"],), generator=g, device=DEV, dtype=torch.int64)
    keys = torch.where(keys >= 1 << 31, keys - (1 << 32), keys).to(torch.int32)
    values = torch.arange(case["n"], dtype=torch.int32, device=DEV)
    return dict(kind=kind, ctx=api.Context(sync=False), bits=case["bits"], keys_in=keys, values_in=values,
                keys=torch.zeros_like(keys), values=torch.zeros_like(values))


def run(s):
    kind = s["kind"]
    if kind == "mono":
        o = s["ctx"].render_dominant(s["scene"], s["cam"], out=s["out"])
        return {k: o[k] for k in ("rgb", "depth_raw", "alpha")}
    if kind == "stereo":
        o = s["ctx"].render_stereo(s["scene"], s["cd"], s["ca"], roi=s["roi"], out=s["out"])
        return {k: v for k, v in o.items() if isinstance(v, torch.Tensor)}
    if kind == "batch":
        with torch.cuda.stream(s["stream"]):
            s["batch"].replay()
        return [{k: o[k] for k in ("rgb_dom", "depth_raw_dom", "alpha_dom", "rgb_aff", "z_aff", "alpha_aff", "cls_aff",
                                   "n_boxes")} for o in s["batch"].outs]
    if kind == "repair":
        s["net"].forward(s["rgb"], s["z"], s["hole"], out=s["out"], err=s["err"])
        return dict(rgb=s["out"], err=s["err"])
    if kind == "train":
        n = s["net"]
        loss = n.train_step(s["rgb"], s["z"], s["hole"], s["target"], lr=2e-3)
        return dict(loss=loss, grad=n.grad, params=n.params, m=n.m, v=n.v)
    if kind == "warp":
        w = s["ctx"].reproject(s["src"], s["dst"], s["rgb"], s["depth"], s["alpha"], s["roi"], out=s["warp"])
        c = s["ctx"].classify_holes(s["src"], s["dst"], w["depth_range"], w["rgb"], w["z"], w["alpha"], w["hole"],
                                    s["roi"], out=s["cls"])
        return dict(w, **c)
    # The sort is in place, so a program writes its new keys first.
    s["keys"].copy_(s["keys_in"])
    s["values"].copy_(s["values_in"])
    keys, values = s["ctx"].sort_pairs(s["keys"], s["values"], s["bits"])
    return dict(keys=keys, values=values)


# --------------------------------------------------------------------------
# What a pass cannot do without.
# --------------------------------------------------------------------------

def _render_work(kind, n, w, h):
    """(scene bytes, flops of one eye): the scene read once; 38 flops per
    contributing (pixel, surfel) pair, about 40 pairs until a pixel is
    opaque, fewer where the surfels' footprints do not cover as much."""
    per = 52 if kind == "cube" else 232
    f_over_z = {"cube": 300.0 * w / 256 / 4, "sphere": 1.375 * w / 2, "unbounded": 1300.0 * w / 1600 / 5}[kind]
    pairs = min(40.0 * w * h, n * 15.0 * 0.0012 * f_over_z * f_over_z)
    return per * n, 38.0 * pairs


def work(case):
    kind = case["kind"]
    if kind == "batch":
        sizes = [max(1000, int(case["scale"] * n)) for n in (50_000, 200_000, 600_000, 1_200_000)]
        total = {"bytes": 0.0, "flops": 0.0}
        for i in range(case["pairs"]):
            w, h = synth.BATCH_RESOLUTIONS[i * 3 % 4]
            b, f = _render_work(("cube", "sphere")[i % 2], sizes[i % 4], w, h)
            total["bytes"] += b + 45 * w * h
            total["flops"] += f
        return total
    if kind == "sort":
        return {"bytes": 16.0 * case["n"], "flops": 0.0}
    px = case["w"] * case["h"]
    if kind in ("mono", "stereo"):
        b, f = _render_work(case["scene"], case["n"], case["w"], case["h"])
        return {"bytes": b + (20 if kind == "mono" else 45) * px, "flops": f}
    if kind == "warp":
        return {"bytes": (41 + 5) * px, "flops": 0.0}
    px *= case["batch"]
    params = repair.num_params()
    if kind == "repair":
        return {"bytes": 33.0 * px + 4 * params, "flops": repair.flops_per_pixel() * px}
    return {"bytes": 29.0 * px + 8 * 4 * params, "flops": 3 * repair.flops_per_pixel() * px}


# --------------------------------------------------------------------------
# The same in 64 bits.
# --------------------------------------------------------------------------

def _sh_basis(d):
    x, y, z = d
    one = torch.ones_like(x)
    pi = math.pi
    c = lambda a, b: math.sqrt(a / (b * pi))  # noqa: E731
    return torch.stack([
        c(1, 4) * one, -c(3, 4) * y, c(3, 4) * z, -c(3, 4) * x,
        c(15, 4) * x * y, -c(15, 4) * y * z, c(5, 16) * (3 * z * z - 1), -c(15, 4) * x * z, c(15, 16) * (x * x - y * y),
        -c(35, 32) * y * (3 * x * x - y * y), c(105, 4) * x * y * z, -c(21, 32) * y * (5 * z * z - 1),
        c(7, 16) * z * (5 * z * z - 3), -c(21, 32) * x * (5 * z * z - 1), c(105, 16) * z * (x * x - y * y),
        -c(35, 32) * x * (x * x - 3 * y * y)])


def _render64(scene, cam, alpha_min=1.0 / 255.0, alpha_max=0.99, t_min=1e-4):
    """Every pixel against every surfel, in depth order."""
    f64 = lambda a: torch.from_numpy(np.asarray(a)).to(DEV, torch.float64)  # noqa: E731
    alpha_min, alpha_max, t_min = (float(np.float32(v)) for v in (alpha_min, alpha_max, t_min))
    R, t = f64(cam.R), f64(cam.t)
    # The order is by centre depth in 32 bits.
    p32 = torch.from_numpy(scene.pos).to(DEV)
    row = R[:, 2].float()
    key = ((row[0] * p32[0] + row[1] * p32[1]) + row[2] * p32[2]) + (-((R[0, 2] * t[0] + R[1, 2] * t[1]) +
                                                                      R[2, 2] * t[2])).float()
    op = f64(scene.opacity)
    live = torch.nonzero((key.double() > cam.z_near) & (op >= alpha_min))[:, 0]
    order = live[torch.sort(key[live], stable=True)[1]]
    pos, q, op = f64(scene.pos)[:, order], f64(scene.quat)[:, order], op[order]
    scale = f64(scene.scale)[:, order]
    q = q / q.norm(dim=0, keepdim=True)
    w, x, y, z = q
    tu = torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y + w * z), 2 * (x * z - w * y)])
    tv = torch.stack([2 * (x * y - w * z), 1 - 2 * (x * x + z * z), 2 * (y * z + w * x)])
    d = pos - t[:, None]
    nc = (scene.sh_degree + 1) ** 2
    sh = f64(scene.sh)[:, order].reshape(nc, 3, -1)
    col = (torch.einsum("kn,kcn->cn", _sh_basis(d / d.norm(dim=0, keepdim=True))[:nc], sh) + 0.5).clamp_min(0.0)
    p, a, b = R.T @ d, R.T @ tu, R.T @ tv
    nv = torch.linalg.cross(a.T, b.T).T
    mux, muy = cam.fx * p[0] / p[2] + cam.cx, cam.fy * p[1] / p[2] + cam.cy
    col1 = lambda v: v[:, None]  # noqa: E731
    h, wd = cam.height, cam.width
    step = max(1, int(4e7) // max(1, order.numel()))
    rgb = torch.empty((3, h * wd), dtype=torch.float64, device=DEV)
    depth, alpha = torch.empty_like(rgb[0]), torch.empty_like(rgb[0])
    for i0 in range(0, h * wd, step):
        idx = torch.arange(i0, min(h * wd, i0 + step), device=DEV)
        py, px = (idx // wd).double(), (idx % wd).double()
        rx, ry = (px - cam.cx) / cam.fx, (py - cam.cy) / cam.fy
        lam = col1((nv * p).sum(0)) / (col1(nv[0]) * rx + col1(nv[1]) * ry + col1(nv[2]))
        hx, hy, hz = lam * rx - col1(p[0]), lam * ry - col1(p[1]), lam - col1(p[2])
        u = (hx * col1(a[0]) + hy * col1(a[1]) + hz * col1(a[2])) / col1(scale[0])
        v = (hx * col1(b[0]) + hy * col1(b[1]) + hz * col1(b[2])) / col1(scale[1])
        e3 = torch.where(lam > cam.z_near, -0.5 * (u * u + v * v), -math.inf)
        e2 = -((px - col1(mux)) ** 2 + (py - col1(muy)) ** 2)
        al = (col1(op) * torch.exp(torch.maximum(e3, e2))).clamp_max(alpha_max)
        al = torch.where(al >= alpha_min, al, 0.0)
        ds = torch.where(e3 >= e2, lam, col1(p[2]).expand_as(lam))
        after = torch.cumprod(1.0 - al, dim=0)
        before = torch.cat([torch.ones_like(after[:1]), after[:-1]])
        wt = torch.where(after >= t_min, al * before, 0.0)
        rgb[:, i0:i0 + step] = col @ wt  # black background
        depth[i0:i0 + step] = (wt * torch.where(wt > 0, ds, 0.0)).sum(0)
        alpha[i0:i0 + step] = wt.sum(0)
    return rgb.reshape(3, h, wd), depth.reshape(h, wd), alpha.reshape(h, wd)


def _conv64(x, weight, bias):
    """3x3 convolution, zero padded, as nine products."""
    b, c, h, w = x.shape
    xp = torch.nn.functional.pad(x, (1, 1, 1, 1))
    out = bias[:, None].expand(-1, b * h * w)
    for k in range(9):
        part = xp[:, :, k // 3:k // 3 + h, k % 3:k % 3 + w].permute(1, 0, 2, 3).reshape(c, -1)
        out = out + weight[:, :, k // 3, k % 3] @ part
    return out.reshape(-1, b, h, w).permute(1, 0, 2, 3)


def _net64(params, rgb, z, hole):
    """The repair network's residual and error channel."""
    m = hole.bool()[:, None]
    inv = torch.where(hole.bool() | torch.isinf(z), 0.0, 1.0 / z.double())
    x = torch.cat([torch.where(m, 0.0, rgb.double()), m.double(), inv[:, None]], dim=1)
    at = 0
    layers = []
    for ci, co in repair.LAYERS:
        wt = params[at:at + co * ci * 9].reshape(co, ci, 3, 3)
        at += co * ci * 9
        layers.append((wt, params[at:at + co]))
        at += co
    pool = lambda v: torch.nn.functional.avg_pool2d(v, 2)  # noqa: E731
    up = lambda v: v.repeat_interleave(2, 2).repeat_interleave(2, 3)  # noqa: E731
    c = lambda v, k: torch.relu(_conv64(v, *layers[k]))  # noqa: E731
    e1 = c(c(x, 0), 1)
    e2 = c(c(pool(e1), 2), 3)
    e3 = c(c(pool(e2), 4), 5)
    d2 = c(torch.cat([up(e3), e2], 1), 6)
    d1 = c(torch.cat([up(d2), e1], 1), 7)
    return _conv64(d1, *layers[8])


def exact(case, seed):
    kind = case["kind"]
    if kind in ("mono", "stereo"):
        if case["n"] * case["w"] * case["h"] > 1e9:
            return None  # every pair would take too long
        cam, _ = _cameras(case["scene"], case["w"], case["h"], case["pose"])
        rgb, depth, alpha = _render64(_scene(case["scene"], case["n"], seed), cam)
        if kind == "mono":
            return dict(rgb=rgb, depth_raw=depth, alpha=alpha)
        return dict(rgb_dom=rgb, depth_raw_dom=depth, alpha_dom=alpha, rgb_aff=None, z_aff=None, alpha_aff=None,
                    cls_aff=None, labels=None, boxes=None, n_boxes=None, tile_mask=None)
    if kind not in ("repair", "train"):
        return None
    rgb, z, hole, target = _warped(seed, case["batch"], case["h"], case["w"])
    params = torch.from_numpy(repair.init_params(seed)).to(DEV, torch.float64)
    m = hole.bool()[:, None]
    if kind == "repair":
        with torch.no_grad():
            r = _net64(params, rgb, z, hole)
        return dict(rgb=rgb.double() + torch.where(m, r[:, :3], 0.0), err=torch.where(m[:, 0], r[:, 3], 0.0))
    params.requires_grad_(True)
    r = _net64(params, rgb, z, hole)
    d = torch.where(m, rgb.double() + r[:, :3] - target.double(), 0.0)
    sq = (d * d).mean(1)
    n = max(1, int(hole.sum()))
    loss = (d * d).sum() / (3 * n) + (torch.where(m[:, 0], r[:, 3] - sq.detach(), 0.0) ** 2).sum() / n
    (grad,) = torch.autograd.grad(loss, params)
    mom, var = 0.1 * grad, 0.001 * grad * grad
    new = params.detach() - 2e-3 * grad / (grad.abs() + 1e-8)
    return dict(loss=loss.detach().reshape(1), grad=grad, params=new, m=mom, v=var)
