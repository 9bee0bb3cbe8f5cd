"""Workloads of the surfel rasterizer for timing: training steps, serving renders, trimming, the densification
action, the photometric loss, the crop volume and the codebook of the serving storage.

Every case runs through the package's public entry points on seeded synthetic scenes (an aerial city for the
large ones, a unit cube of surfels for the small ones) drawn on the GPU.  ``exact`` gives the results of the
cases small enough for it in float64, by brute force over every (pixel, surfel) pair in plain torch.
"""
import math

import numpy as np
import torch

from paper_2411_00771_amd import crop, raster, scenes, server, storage

DEV = "cuda"
PAIRS = 1_500_000_000  # (pixel, surfel) pairs and (point, view) pairs the float64 results are computed for


def listed():
    step = dict(kind="step", views=1, degree=3, geometry=False, elongated=0.05, city=True)
    view = dict(kind="render", n=5_000_000, views=1, compact=False, degree=3)
    return [
        # one small view of a few thousand surfels: start of training, unit scenes, interactive edits; launches
        dict(step, name="step-4k-128", n=4096, width=128, height=128, city=False),
        # the autograd form with depth, normal and opacity terms in the loss, ragged image and surfel count
        dict(step, name="step-autograd-23k-317x203", n=23_001, width=317, height=203, degree=1, geometry=True,
             city=False),
        # the training step of an aerial block: one image of the paper's size against 1 M surfels
        dict(step, name="step-1m-1600x1066", n=1_000_000, width=1600, height=1066),
        # the largest training launch: 8 views per call, 10 M surfels, a tenth of them long and thin
        dict(step, name="step-10m-8v-1600x1066", n=10_000_000, views=8, width=1600, height=1066, elongated=0.1),
        # serving a small preview of a large scene: the projection and the binning dominate
        dict(view, name="render-5m-640x480", width=640, height=480),
        # serving 4K views from the compact storage (SH degree 2, float16, codebook)
        dict(view, name="render-5m-compact-3840x2160", width=3840, height=2160, compact=True, degree=2),
        # a burst of mixed-resolution requests through the render server
        dict(kind="serve", name="serve-5m-burst12", n=5_000_000, requests=12, slots=4, batch=1, degree=3),
        # contribution-based trimming over the views of a block, and its percentile mask
        dict(kind="trim", name="trim-1m-4v-1600x1066", n=1_000_000, width=1600, height=1066, views=4, degree=3,
             city=True, ratio=0.025, gamma=0.5),
        # the densification action every few hundred steps, with the optimiser's moments re-laid
        dict(kind="action", name="action-1m", n=1_000_000, degree=3, candidates=0.05, removed=0.025),
        # the photometric loss alone on ragged images
        dict(kind="loss", name="loss-3v-1237x823", views=3, width=1237, height=823),
        # the crop volume of the evaluation protocol at the scale it is quoted on
        dict(kind="crop", name="crop-31m-958v", points=31_400_000, views=958, width=1920, height=1080, tau=3),
        # one Lloyd iteration of the serving codebook (40 % of 1 M surfels, degree 2)
        dict(kind="lloyd", name="lloyd-400k-8192x27", rows=400_000, codewords=8192, degree=2),
    ]


def _between(rng, a, b):
    """An integer of [a, b], its logarithm uniform."""
    return max(a, min(b, int(round(math.exp(rng.uniform(math.log(a), math.log(b)))))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "step", "render", "render", "serve", "trim", "action", "loss", "crop",
                       "lloyd"])
    width = _between(rng, 97, 1920)
    height = max(64, int(width * rng.uniform(0.5, 0.9)))
    degree = rng.randrange(4)
    if kind == "step":
        n = _between(rng, 3000, 5_000_000)
        views = rng.choice([1, 1, 1, 2, 3, 5, 8])
        while n * views > 16_000_000 or width * height * views > 8_000_000:
            views -= 1
        city = n > 50_000
        return dict(kind=kind, n=n, views=views, width=width, height=height, degree=degree,
                    geometry=rng.random() < 0.3, elongated=rng.choice([0.05, 0.1]), city=city)
    if kind == "render":
        width = _between(rng, 240, 3840)
        compact = rng.random() < 0.5
        return dict(kind=kind, n=_between(rng, 60_000, 8_000_000), views=rng.choice([1, 1, 2]), width=width,
                    height=int(width * rng.uniform(0.5, 0.8)), compact=compact, degree=2 if compact else degree)
    if kind == "serve":
        return dict(kind=kind, n=_between(rng, 300_000, 5_000_000), requests=rng.randrange(4, 17),
                    slots=rng.choice([1, 2, 4]), batch=rng.choice([1, 2, 4]), degree=degree)
    if kind == "trim":
        n = _between(rng, 3000, 3_000_000)
        return dict(kind=kind, n=n, width=width, height=height, views=rng.randrange(1, 6), degree=degree,
                    city=n > 50_000, ratio=rng.choice([0.025, 0.1, 0.4]), gamma=rng.choice([0.5, 0.5, 0.3]))
    if kind == "action":
        return dict(kind=kind, n=_between(rng, 3000, 5_000_000), degree=degree,
                    candidates=round(rng.uniform(0.01, 0.2), 3), removed=round(rng.uniform(0.0, 0.5), 3))
    if kind == "loss":
        return dict(kind=kind, views=rng.randrange(1, 9), width=width, height=height)
    if kind == "crop":
        return dict(kind=kind, points=_between(rng, 30_000, 20_000_000), views=_between(rng, 16, 900), width=1920,
                    height=1080, tau=rng.randrange(1, 6))
    rows = _between(rng, 5000, 400_000)
    return dict(kind="lloyd", rows=rows, codewords=min(rows, rng.choice([256, 1024, 4096, 8191, 8192])),
                degree=rng.choice([1, 2, 3]))


# ---- inputs ------------------------------------------------------------------------------------------


def _rand(g, *shape):
    return torch.rand(shape, device=DEV, generator=g)


def _randn(g, *shape):
    return torch.randn(shape, device=DEV, generator=g)


def _gen(seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    return g


def _colour(g, n, degree):
    sh = 0.05 * _randn(g, n, (degree + 1) ** 2, 3)
    sh[:, 0] = _rand(g, n, 3)
    return sh


def _cloud(seed, n, degree):
    """Surfels of random orientation in the cube [-1, 1]^3."""
    g = _gen(seed)
    lo, hi = math.log(0.005), math.log(0.05)
    quat = _randn(g, 4, n)
    return raster.Params(2 * _rand(g, 3, n) - 1, lo + (hi - lo) * _rand(g, 2, n), quat / quat.norm(dim=0),
                         _randn(g, n), _colour(g, n, degree), degree)


def _surface(g, city, n):
    """Points [n][3] (float64) and normals on the city's terrain, roofs and walls, area-proportional."""
    B = torch.from_numpy(city.boxes).to(DEV)
    roof = B[:, 2] * B[:, 3]
    faces = torch.stack([B[:, 3] * B[:, 4], B[:, 3] * B[:, 4], B[:, 2] * B[:, 4], B[:, 2] * B[:, 4]], 1).reshape(-1)
    areas = torch.cat([torch.tensor([city.L ** 2], device=DEV, dtype=torch.float64), roof, faces])
    edges = torch.cumsum(areas, 0)
    pick = torch.searchsorted(edges, torch.rand(n, device=DEV, generator=g, dtype=torch.float64) * edges[-1])
    pick = pick.clamp_(max=len(areas) - 1)
    u = torch.rand(2, n, device=DEV, generator=g, dtype=torch.float64) - 0.5
    # terrain: the height field and its gradient
    x, y = u[0] * city.L, u[1] * city.L
    z, gx, gy = torch.zeros_like(x), torch.zeros_like(x), torch.zeros_like(x)
    for amp, lam, dirs, ph in city.octaves:
        for d, p in zip(dirs, ph):
            a = 2 * math.pi / lam * (d[0] * x + d[1] * y) + p
            z += amp / math.sqrt(len(dirs)) * torch.sin(a)
            s = amp / math.sqrt(len(dirs)) * 2 * math.pi / lam * torch.cos(a)
            gx += d[0] * s
            gy += d[1] * s
    pos = torch.stack([x, y, z], 1)
    nrm = torch.nn.functional.normalize(torch.stack([-gx, -gy, torch.ones_like(gx)], 1), dim=1)
    # roofs, then the four walls of each box
    nb = len(B)
    box = B[torch.where(pick <= nb, pick - 1, (pick - 1 - nb) // 4).clamp_(min=0)]
    is_roof, is_wall = (pick >= 1) & (pick <= nb), pick > nb
    top = torch.stack([box[:, 0] + u[0] * box[:, 2], box[:, 1] + u[1] * box[:, 3], box[:, 5] + box[:, 4]], 1)
    face = (pick - 1 - nb) % 4
    sx = torch.where(face == 0, 0.5, torch.where(face == 1, -0.5, u[0]))
    sy = torch.where(face == 2, 0.5, torch.where(face == 3, -0.5, u[0]))
    wall = torch.stack([box[:, 0] + sx * box[:, 2], box[:, 1] + sy * box[:, 3],
                        box[:, 5] + (u[1] + 0.5) * box[:, 4]], 1)
    out = torch.tensor([[1.0, 0, 0], [-1.0, 0, 0], [0, 1.0, 0], [0, -1.0, 0]], device=DEV, dtype=torch.float64)
    pos = torch.where(is_roof[:, None], top, torch.where(is_wall[:, None], wall, pos))
    up = torch.tensor([0.0, 0, 1.0], device=DEV, dtype=torch.float64)
    nrm = torch.where(is_roof[:, None], up, torch.where(is_wall[:, None], out[face.clamp(min=0)], nrm))
    return pos, nrm, math.sqrt(float(edges[-1]) / n)


def _city_surfels(seed, city, n, degree, elongated):
    """A trained aerial set: surfels on the surfaces, spacing-sized, a share of them long and thin (the larger
    share with axis ratios up to 1000)."""
    g = _gen(seed)
    mean = torch.empty(3, n, device=DEV)
    quat = torch.empty(4, n, device=DEV)
    spacing = None
    for a in range(0, n, 4_000_000):
        k = min(4_000_000, n - a)
        pos, nrm, sp = _surface(g, city, k)
        spacing = sp * math.sqrt(k / n)
        mean[:, a:a + k] = pos.T
        # the shortest rotation of z onto the normal, after a uniform turn about z
        t = math.pi * torch.rand(k, device=DEV, generator=g, dtype=torch.float64)
        c, s = torch.cos(t), torch.sin(t)
        w, x, y = 1 + nrm[:, 2], -nrm[:, 1], nrm[:, 0]
        q = torch.stack([w * c, x * c + y * s, y * c - x * s, w * s])
        quat[:, a:a + k] = q / q.norm(dim=0)
    if elongated > 0.05:
        ls = math.log(spacing) + 0.6 * _randn(g, 2, n)
        ratio = 50 + 950 * _rand(g, n)
    else:
        ls = torch.log(spacing * (0.5 + _rand(g, 2, n)))
        ratio = 20 + 30 * _rand(g, n)
    long = _rand(g, n) < elongated
    mid, half = 0.5 * (ls[0] + ls[1]), 0.5 * torch.log(ratio)
    ls = torch.stack([torch.where(long, mid + half, ls[0]), torch.where(long, mid - half, ls[1])])
    return raster.Params(mean, ls, quat, _randn(g, n), _colour(g, n, degree), degree)


def _scene(case, seed):
    """(surfels, cameras) of a training or trimming case."""
    if not case["city"]:
        cams = [scenes.tiny_camera(case["width"], case["height"], dist=3.0 + 0.2 * v) for v in range(case["views"])]
        return _cloud(seed, case["n"], case["degree"]), cams
    city = scenes.make_city(seed % 1000)
    p = _city_surfels(seed, city, case["n"], case["degree"], case.get("elongated", 0.05))
    cams = scenes.aerial_cameras(seed + 1000, city, count=case["views"], width=case["width"], height=case["height"])
    return p, cams


def _image(g, views, width, height):
    """Images with structure at all scales, like photographs."""
    img = torch.zeros(views, 3, height, width, device=DEV)
    for k, amp in ((6, 0.5), (24, 0.3), (96, 0.15)):
        low = _rand(g, views, 3, max(2, k * height // width), k)
        img += amp * torch.nn.functional.interpolate(low, size=(height, width), mode="bilinear")
    return (img + 0.05 * _rand(g, views, 3, height, width)).contiguous()


def _engine(params, cams, backward):
    eng = raster.Engine(params.n, cams[0].width, cams[0].height, len(cams), capacity=1 << 20, backward=backward)
    arr = eng.cams(cams)
    eng.fit_capacity(params, arr)
    return eng, arr


def prepare(case, seed):
    g = _gen(seed + 77)
    kind = case["kind"]
    if kind == "step":
        p, cams = _scene(case, seed)
        eng, arr = _engine(p, cams, True)
        s = dict(case=case, eng=eng, cams=arr, params=p, state=raster.DensifyState(p.n, len(cams)),
                 target=_image(g, len(cams), case["width"], case["height"]))
        if case["geometry"]:
            s["leaves"] = [t.requires_grad_(True) for t in (p.mean, p.log_scale, p.quat, p.opacity_logit, p.sh)]
            px = case["width"] * case["height"]
            up = _randn(g, len(cams), 5, case["height"], case["width"]) / px
            s["w_depth"], s["w_normal"] = 0.1 * up[:, 0].contiguous(), 0.05 * up[:, 1:4].contiguous()
            s["w_alpha"] = 0.1 * up[:, 4].contiguous()
        else:
            s["grads"] = raster.Grads(p, len(cams))
        return s
    if kind == "render":
        city = scenes.make_city(seed % 1000, L=1600.0)
        p = _city_surfels(seed, city, case["n"], case["degree"], 0.05)
        rng = np.random.default_rng(seed)
        cams = [scenes.orbit_camera(rng, city, case["width"], case["height"]) for _ in range(case["views"])]
        if case["compact"]:
            p, _ = storage.compress(p, _rand(g, p.n), ratio=0.4, codebook_size=min(8192, p.n // 8), iters=1)
        eng, arr = _engine(p, cams, False)
        return dict(case=case, eng=eng, cams=arr, params=p)
    if kind == "serve":
        city = scenes.make_city(seed % 1000, L=1600.0)
        p = _city_surfels(seed, city, case["n"], case["degree"], 0.05)
        rng = np.random.default_rng(seed)
        res = [scenes.SERVE_RESOLUTIONS[k % 4] for k in range(case["requests"])]
        cams = [scenes.orbit_camera(rng, city, w, h) for w, h in res]
        srv = server.Server(p, max_slots=case["slots"], max_batch=case["batch"], arena_bytes=32 << 30)
        return dict(case=case, server=srv, cams=cams)
    if kind == "trim":
        p, cams = _scene(case, seed)
        one, arrs = None, []
        for c in cams:  # one engine, one view per call, sized for every view
            if one is None:
                one, arr = _engine(p, [c], False)
            else:
                arr = one.cams([c])
                one.fit_capacity(p, arr)
            arrs.append(arr)
        return dict(case=case, eng=one, cams=arrs, params=p, c_sum=torch.zeros(p.n, device=DEV),
                    c_view=torch.empty(len(cams), 1, p.n, device=DEV))
    if kind == "action":
        n = case["n"]
        p = _city_surfels(seed, scenes.make_city(seed % 1000), n, case["degree"], 0.05)
        p.opacity_logit.clamp_(min=-5.0)  # above the removal threshold on opacity
        # disjoint candidates and removals (every candidate adds one surfel to the set, cloned or split)
        pick = torch.randperm(n, device=DEV, generator=g)
        nc, nr = int(n * case["candidates"]), int(n * case["removed"])
        mask = torch.randint(0, 4, (n,), device=DEV, generator=g, dtype=torch.uint8)
        mask[pick[:nc]] |= 4
        remove = torch.zeros(n, device=DEV, dtype=torch.uint8)
        remove[pick[nc:nc + nr]] = 1
        z = _randn(g, n, 2, 2)
        scale = float(torch.exp(p.log_scale.max(0).values).median())
        moments = [[_randn(g, *t.shape) for t in (p.mean, p.log_scale, p.quat, p.opacity_logit, p.sh)]
                   for _ in range(2)]
        return dict(case=case, params=p, mask=mask, remove=remove, z=z, scale=scale, moments=moments)
    if kind == "loss":
        eng = raster.Engine(1, case["width"], case["height"], case["views"], capacity=64)
        target = _image(g, case["views"], case["width"], case["height"])
        img = target + 0.1 * (_image(g, case["views"], case["width"], case["height"]) - 0.5)
        return dict(case=case, eng=eng, target=target, img=img.contiguous())
    if kind == "crop":
        city = scenes.make_city(seed % 1000, L=1212.0)
        pts = torch.empty(3, case["points"], device=DEV)
        for a in range(0, case["points"], 4_000_000):
            k = min(4_000_000, case["points"] - a)
            pos, _, spacing = _surface(g, city, k)
            pts[:, a:a + k] = pos.T + 0.05 * _randn(g, 3, k)
        spacing *= math.sqrt(k / case["points"])
        pts = pts[:, _octree_order(pts)].contiguous()
        cams = scenes.aerial_cameras(seed + 1000, city, count=case["views"], width=case["width"],
                                     height=case["height"])
        T = np.concatenate([np.linalg.qr(np.random.default_rng(seed).normal(size=(3, 3)))[0],
                            np.array([[3.0], [-2.0], [1.0]])], 1)
        return dict(case=case, points=pts, cams=cams, radius=3 * spacing, T=T,
                    outline=torch.zeros(2, case["points"], device=DEV, dtype=torch.float64))
    D = 3 * (case["degree"] + 1) ** 2
    n = case["rows"] * 5 // 2
    x = _colour(g, n, case["degree"]).reshape(n, D)
    rows = torch.randperm(n, device=DEV, generator=g)[:case["rows"]].sort().values.to(torch.int32)
    return dict(case=case, x=x, D=D, rows=rows, start=storage.vq_init(x, D, rows, case["codewords"]))


def _octree_order(pts, bits=21):
    """The permutation into 3-D Morton order, in which octree-indexed point clouds are stored."""
    lo = pts.min(1, keepdim=True).values
    q = ((pts - lo) / (pts - lo).max() * ((1 << bits) - 1)).to(torch.int64)
    code = torch.zeros_like(q[0])
    for b in range(bits):
        for d in range(3):
            code |= ((q[d] >> b) & 1) << (3 * b + d)
    return torch.argsort(code)


# ---- passes ------------------------------------------------------------------------------------------


def run(state):
    return _RUN[state["case"]["kind"]](state)


def _run_step(s):
    eng, st = s["eng"], s["state"]
    if "leaves" in s:
        for t in s["leaves"]:
            t.grad = None
        rgb, depth, dmed, normal, alpha = raster.rasterize(s["leaves"], eng, s["cams"], s["case"]["degree"])
        loss = raster.L1SSIMLoss.apply(rgb, s["target"], eng, raster.LAMBDA_SSIM)
        total = loss + (depth * s["w_depth"]).sum() + (normal * s["w_normal"]).sum() + (alpha * s["w_alpha"]).sum()
        total.backward()
        g = eng.grads
        grads = [t.grad for t in s["leaves"]]
    else:
        g = s["grads"]
        g.zero_()
        eng.forward(s["params"], s["cams"])
        eng.loss(s["target"])
        eng.backward(s["params"], s["cams"], g, d_rgb=eng.d_img, d_rgb_ssim=eng.d_img_ssim)
        grads = [g.mean, g.log_scale, g.quat, g.opacity_logit, g.sh]
    eng.densify(s["params"], g, st)
    return dict(rgb=eng.rgb, depth=eng.depth, depth_med=eng.depth_med, normal=eng.normal, alpha=eng.alpha,
                loss=eng.loss_val, grads=grads, view_total=g.g_view_total, view_ssim=g.g_view_ssim,
                dgd=st.accum_dgd, total=st.accum_total, radius=st.max_radius, denom=st.denom, mask=st.mask,
                scale=st.scale)


def _run_render(s):
    s["eng"].forward(s["params"], s["cams"])
    return dict(rgb=s["eng"].rgb, depth=s["eng"].depth, normal=s["eng"].normal)


def _run_serve(s):
    reqs = [s["server"].submit(c) for c in s["cams"]]
    s["server"].drain()
    s["server"].finished.clear()
    return [r.result for r in reqs]


def _run_trim(s):
    eng, case = s["eng"], s["case"]
    s["c_sum"].zero_()
    for v, arr in enumerate(s["cams"]):
        eng.project(s["params"], arr)
        eng.bin_sort(arr)
        eng.contribution(arr, case["gamma"], c_view=s["c_view"][v], c_sum=s["c_sum"])
    c_avg = s["c_sum"] / len(s["cams"])
    bound, mask, removed = raster.trim_mask(c_avg, case["ratio"])
    return dict(c_view=s["c_view"], c_avg=c_avg, bound=bound, mask=mask, removed=removed)


def _run_action(s):
    p = s["params"]
    plan = raster.densify_plan(p, s["mask"], s["remove"], dense_scale=s["scale"])
    out, src = raster.densify_apply(p, plan, s["z"])
    moments = [[raster.densify_gather(t, src, plan, out.n, blocked=k == 4, zero_new=True) for k, t in enumerate(m)]
               for m in s["moments"]]
    return dict(actions=plan.actions, counts=plan.counts, src=src, moments=moments,
                out=[out.mean, out.log_scale, out.quat, out.opacity_logit, out.sh])


def _run_loss(s):
    eng = s["eng"]
    return dict(loss=eng.loss(s["target"], img=s["img"]), d_img=eng.d_img, d_img_ssim=eng.d_img_ssim)


def _run_crop(s):
    count = crop.visibility_count(s["points"], s["cams"], s["radius"], 2.1213)
    keep, ground, (lo, hi) = crop.crop_volume(s["points"], count, s["case"]["tau"], s["T"])
    s["outline"][:, :ground.shape[1]] = ground  # kept for the alpha shape
    return dict(count=count, keep=keep, ground=s["outline"], low=lo, high=hi)


def _run_lloyd(s):
    cb = s["start"].clone()
    code = storage.vq_assign(s["x"], s["D"], s["rows"], cb)
    counts = storage.vq_update(s["x"], s["D"], s["rows"], code, cb)
    return dict(code=code, codebook=cb, counts=counts)


_RUN = dict(step=_run_step, render=_run_render, serve=_run_serve, trim=_run_trim, action=_run_action, loss=_run_loss,
            crop=_run_crop, lloyd=_run_lloyd)


# ---- work and tolerances -----------------------------------------------------------------------------

# Per pixel of an aerial view: about 100 list entries are evaluated (35 flops each: the ray-splat intersection,
# the filter and the Gaussian), half of them blended (21 flops forward, 151 in the reverse pass, 7 for a
# contribution); about 8 % of the surfels are visible in a view and read their colour.
EVAL, BLEND = 100, 50


def work(case):
    kind = case["kind"]
    if kind in ("loss", "step", "render", "trim"):
        px = case["views"] * case["width"] * case["height"]
    if kind == "loss":
        return dict(bytes=4.0 * px * 12, flops=px * 3 * 4 * 11 * 4.0)
    if kind in ("step", "render", "trim"):
        n, v, deg = case["n"], case["views"], case["degree"]
        sh = 12 * (deg + 1) ** 2
        seen = 0.08 if case.get("city", True) else 1.0
        if case.get("compact"):
            params = n * (12 + 14 + seen * v * sh / 2)
        else:
            params = n * (40 + min(1.0, seen * v) * sh)
        if kind == "render":
            return dict(bytes=params + 28.0 * px, flops=px * (EVAL * 35.0 + BLEND * 21) + n * v * 200.0)
        if kind == "trim":
            return dict(bytes=params + 4.0 * n * v + 9.0 * n, flops=px * (EVAL * 35.0 + BLEND * 7) + n * v * 200.0)
        grads = n * (40 + sh) + 16.0 * n * v
        images = px * (36.0 + 12 + (20 if case["geometry"] else 0))
        return dict(bytes=params + grads + images + 33.0 * n,
                    flops=px * (2 * EVAL * 35.0 + BLEND * 172 + 600) + n * v * 200.0)
    if kind == "serve":
        px = sum(w * h for w, h in (scenes.SERVE_RESOLUTIONS[k % 4] for k in range(case["requests"])))
        sh = 12 * (case["degree"] + 1) ** 2
        return dict(bytes=case["requests"] * case["n"] * (40 + 0.08 * sh) + 28.0 * px,
                    flops=px * (EVAL * 35.0 + BLEND * 21) + case["n"] * case["requests"] * 200.0)
    if kind == "action":
        row = 40 + 12 * (case["degree"] + 1) ** 2
        kept = 1 - case["removed"]
        return dict(bytes=case["n"] * (2 + 3 * row * (kept + kept + case["candidates"]) + 12), flops=100.0 * case["n"])
    if kind == "crop":
        # the decisions of a view whose edge crosses a point's neighbourhood are taken point by point
        return dict(bytes=case["points"] * (12 + 4 + 1 + 16.0), flops=case["points"] * (case["views"] * 2.0 + 40))
    D = 3 * (case["degree"] + 1) ** 2
    return dict(bytes=4.0 * D * (case["rows"] + 2 * case["codewords"]) + 6.0 * case["rows"],
                flops=2.0 * case["rows"] * case["codewords"] * D)


def tolerance(case):
    return _TOLERANCE[case["kind"]]


# Four times what float32 sums in another order and the float64 results show: the gradients are added with atomics
# (two passes over the same inputs differ by 7e-6, single elongated surfels by 2e-3 of their value), the densification
# gradients are 1e-4 off float64, the SSIM gradient 8.5e-5 (the variances cancel), the codebook 2.6e-4 (near ties).
_TOLERANCE = dict(step={"rel": 4e-4, "max": 0.1, "differ": 1e-4}, render={"rel": 1e-4, "max": 0.1},
                  serve={"rel": 1e-4, "max": 0.1}, trim={"rel": 1e-5, "max": 1e-2, "differ": 1e-4},
                  action="exact", loss={"rel": 3.4e-4, "max": 0.05}, crop={"rel": 1e-13, "max": 1e-12},
                  lloyd={"rel": 1e-3, "max": 0.1, "differ": 4e-3})


# ---- float64 results ---------------------------------------------------------------------------------


def exact(case, seed):
    kind = case["kind"]
    if kind in ("step", "trim"):
        if case["n"] * case["views"] * case["width"] * case["height"] > PAIRS:
            return None
    if kind == "crop" and case["points"] * case["views"] > 2 * PAIRS:
        return None
    if kind in ("serve", "render"):  # large scenes only
        return None
    f = dict(step=_exact_step, trim=_exact_trim, action=_exact_action, loss=_exact_loss, crop=_exact_crop,
             lloyd=_exact_lloyd)[kind]
    return f(case, prepare(case, seed))


def _rotation(q):
    w, x, y, z = q / q.norm(dim=0)
    return torch.stack([torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y)]),
                        torch.stack([2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x)]),
                        torch.stack([2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)])])


def _harmonics(degree, d):
    """Real spherical harmonics with the Condon-Shortley phase at unit directions d [3][n]: [K][n]."""
    x, y, z = d
    c = [math.sqrt(1 / (4 * math.pi)), math.sqrt(3 / (4 * math.pi)), math.sqrt(15 / (4 * math.pi)),
         math.sqrt(5 / (16 * math.pi)), math.sqrt(35 / (32 * math.pi)), math.sqrt(105 / (4 * math.pi)),
         math.sqrt(21 / (32 * math.pi)), math.sqrt(7 / (16 * math.pi))]
    Y = [c[0] * torch.ones_like(x)]
    if degree > 0:
        Y += [-c[1] * y, c[1] * z, -c[1] * x]
    if degree > 1:
        Y += [c[2] * x * y, -c[2] * y * z, c[3] * (3 * z * z - 1), -c[2] * x * z, 0.5 * c[2] * (x * x - y * y)]
    if degree > 2:
        Y += [-c[4] * y * (3 * x * x - y * y), c[5] * x * y * z, -c[6] * y * (5 * z * z - 1),
              c[7] * z * (5 * z * z - 3), -c[6] * x * (5 * z * z - 1), 0.5 * c[5] * z * (x * x - y * y),
              -c[4] * x * (x * x - 3 * y * y)]
    return torch.stack(Y)


class _View:
    """One view's surfels in float64, front to back, with the shift of their screen image as a variable."""

    def __init__(self, leaves, degree, cam):
        mean, ls, quat, logit, sh = leaves
        f64 = dict(device=DEV, dtype=torch.float64)
        R = torch.tensor(np.float32(cam.R), **f64)
        t = torch.tensor(np.float32(cam.t), **f64)
        fx, fy, cx, cy = (float(np.float32(k)) for k in (cam.fx, cam.fy, cam.cx, cam.cy))
        n = mean.shape[1]
        self.shift = torch.zeros(2, n, requires_grad=True, **f64)
        s, o = torch.exp(ls), torch.sigmoid(logit)
        frame = torch.einsum("ij,jkn->ikn", R, _rotation(quat))
        pc = R @ mean + t[:, None]
        cols = torch.stack([frame[:, 0] * s[0], frame[:, 1] * s[1], pc], 1)  # [3 rows][3 columns][n]
        m3 = cols[2]
        m1 = fx * cols[0] + cx * m3 + self.shift[0] * m3
        m2 = fy * cols[1] + cy * m3 + self.shift[1] * m3
        flip = torch.where((frame[:, 2] * pc).sum(0) > 0, -1.0, 1.0).detach()
        view = mean + (R.T @ t)[:, None]
        Y = _harmonics(degree, view / view.norm(dim=0))
        rgb = torch.relu(0.5 + torch.einsum("kn,nkc->cn", Y, sh))
        k2 = 2 * torch.log(255 * o)
        ok = (pc[2] > float(np.float32(cam.znear))) & (k2 > 0)
        ok &= m3[0] ** 2 + m3[1] ** 2 - m3[2] ** 2 / k2.clamp(min=1e-300) < 0
        ids = ok.nonzero().reshape(-1)
        ids = ids[torch.sort(pc[2].detach()[ids].float(), stable=True).indices]
        self.ids, self.n = ids, n
        self.m1, self.m2, self.m3, self.o = m1[:, ids], m2[:, ids], m3[:, ids], o[ids]
        self.attr = torch.cat([rgb, flip * frame[:, 2]])[:, ids]
        self.chunk = max(1, 3_000_000 // max(1, len(ids)))

    def pixels(self, px, py):
        """(weights, alpha, T in front, depth, T at the end) of the sorted surfels at pixels (px, py)."""
        x, y = px[:, None] + 0.5, py[:, None] + 0.5
        a = [x * self.m3[k] - self.m1[k] for k in range(3)]
        b = [y * self.m3[k] - self.m2[k] for k in range(3)]
        p = [a[1] * b[2] - a[2] * b[1], a[2] * b[0] - a[0] * b[2], a[0] * b[1] - a[1] * b[0]]
        w = torch.where(p[2] == 0, torch.full_like(p[2], 1e-300), p[2])
        u, v = p[0] / w, p[1] / w
        r3 = u * u + v * v
        r2 = 2 * ((x - self.m1[2] / self.m3[2]) ** 2 + (y - self.m2[2] / self.m3[2]) ** 2)
        is3 = r3 <= r2
        rho = torch.where(is3, r3, r2)
        z = torch.where(is3, self.m3[0] * u + self.m3[1] * v + self.m3[2], self.m3[2].expand_as(u))
        alpha = (self.o * torch.exp(-0.5 * rho)).clamp(max=0.99)
        alpha = torch.where(alpha >= 1 / 255, alpha, torch.zeros_like(alpha))
        after = torch.exp(torch.cumsum(torch.log1p(-alpha), 1))
        alpha = torch.where(after.detach() >= 1e-4, alpha, torch.zeros_like(alpha))
        logT = torch.cumsum(torch.log1p(-alpha), 1)
        front = torch.exp(logT - torch.log1p(-alpha))
        return alpha * front, alpha, front, z, torch.exp(logT[:, -1])

    def blend(self, px, py):
        """[8][pixels]: colour, normal, depth, alpha; and the median depth."""
        w, alpha, front, z, T = self.pixels(px, py)
        out = torch.cat([torch.einsum("pn,cn->cp", w, self.attr), (w * z).sum(1)[None], (1 - T)[None]])
        pick = (alpha > 0) & (front > 0.5)
        last = (pick * torch.arange(1, pick.shape[1] + 1, device=DEV)).max(1).values
        med = torch.where(last > 0, z.gather(1, (last - 1).clamp(min=0)[:, None])[:, 0], torch.zeros_like(T))
        return out, med


def _chunks(cam, size):
    total = cam.width * cam.height
    for a in range(0, total, size):
        k = torch.arange(a, min(total, a + size), device=DEV)
        yield a, (k % cam.width).double(), (k // cam.width).double()


def _window_sum(x):
    g = torch.exp(-torch.arange(-5, 6, device=DEV, dtype=torch.float64) ** 2 / (2 * 1.5 ** 2))
    g = g / g.sum()
    for dim in (-1, -2):
        pad = (5, 5, 0, 0) if dim == -1 else (0, 0, 5, 5)
        p = torch.nn.functional.pad(x, pad)
        x = sum(g[k] * p.narrow(dim, k, x.shape[dim]) for k in range(11))
    return x


def _loss64(img, target, lam=raster.LAMBDA_SSIM):
    """(loss [V][3], d loss / d img, its SSIM part) per view."""
    x, y = img.detach().double().requires_grad_(True), target.double()
    mx, my = _window_sum(x), _window_sum(y)
    sxx, syy, sxy = _window_sum(x * x) - mx * mx, _window_sum(y * y) - my * my, _window_sum(x * y) - mx * my
    ssim = ((2 * mx * my + 1e-4) * (2 * sxy + 9e-4)) / ((mx * mx + my * my + 1e-4) * (sxx + syy + 9e-4))
    ssim, l1 = ssim.mean((1, 2, 3)), (x - y).abs().mean((1, 2, 3))
    ds = torch.autograd.grad((lam * (1 - ssim)).sum(), x, retain_graph=True)[0]
    d1 = torch.autograd.grad(((1 - lam) * l1).sum(), x)[0]
    return torch.stack([(1 - lam) * l1 + lam * (1 - ssim), l1, ssim], 1).detach(), ds + d1, ds


def _leaves64(p):
    return [t.detach().double().requires_grad_(True) for t in (p.mean, p.log_scale, p.quat, p.opacity_logit, p.sh)]


def _exact_step(case, s):
    cams = _cameras(s["cams"])
    leaves = _leaves64(s["params"])
    W, H, V = case["width"], case["height"], case["views"]
    img = torch.zeros(V, 8, H * W, device=DEV, dtype=torch.float64)
    med = torch.zeros(V, H * W, device=DEV, dtype=torch.float64)
    views = []
    for v, cam in enumerate(cams):
        with torch.no_grad():
            view = _View(leaves, case["degree"], cam)
            for a, px, py in _chunks(cam, view.chunk):
                img[v, :, a:a + len(px)], med[v, a:a + len(px)] = view.blend(px, py)
    img = img.view(V, 8, H, W)
    loss, d_img, d_ssim = _loss64(img[:, :3], s["target"])
    up = torch.zeros(V, 8, H, W, device=DEV, dtype=torch.float64)
    up[:, :3] = d_img
    if case["geometry"]:
        up[:, 3:6], up[:, 6], up[:, 7] = s["w_normal"].double(), s["w_depth"].double(), s["w_alpha"].double()
    vt = torch.zeros(V, 2, case["n"], device=DEV, dtype=torch.float64)
    vs = torch.zeros_like(vt)
    for v, cam in enumerate(cams):
        proto = _View(leaves, case["degree"], cam)
        # the pixels' gradients with respect to the sorted surfels, then one chain back to the parameters
        fields = ("m1", "m2", "m3", "o", "attr")
        cut = [getattr(proto, k).detach().requires_grad_(True) for k in fields]
        for k, t in zip(fields, cut):
            setattr(proto, k, t)
        acc, acc_s = [torch.zeros_like(t) for t in cut], [torch.zeros_like(t) for t in cut]
        for a, px, py in _chunks(cam, proto.chunk):
            out, _ = proto.blend(px, py)
            u = up[v].reshape(8, -1)[:, a:a + len(px)]
            us = d_ssim[v].reshape(3, -1)[:, a:a + len(px)]
            for t, g in zip(acc, torch.autograd.grad((out * u).sum(), cut, retain_graph=True)):
                t += g
            for t, g in zip(acc_s, torch.autograd.grad((out[:3] * us).sum(), cut, allow_unused=True)):
                t += 0 if g is None else g
        full = _View(leaves, case["degree"], cam)
        roots = [getattr(full, k) for k in fields]
        vs[v] = torch.autograd.grad(roots, full.shift, acc_s, retain_graph=True, allow_unused=True)[0]
        got = torch.autograd.grad(roots, leaves + [full.shift], acc)
        vt[v] = got[5]
        for t, g in zip(leaves, got):
            t.grad = g if t.grad is None else t.grad + g
    half = torch.tensor([W / 2, H / 2], device=DEV, dtype=torch.float64)[None, :, None]
    vt, vs = vt * half, vs * half
    nt, ns = vt.norm(dim=1), vs.norm(dim=1)
    scale = torch.clamp(0.9 * nt.sum(1) / ns.sum(1).clamp(min=1e-300), min=1.0)
    return dict(rgb=img[:, :3], depth=img[:, 6], depth_med=None, normal=img[:, 3:6], alpha=img[:, 7], loss=loss,
                grads=[t.grad for t in leaves], view_total=vt, view_ssim=vs, dgd=(scale[:, None] * ns).sum(0),
                total=nt.sum(0), radius=None, denom=None, mask=None, scale=scale)


def _cameras(arr):
    """Cameras with the attributes of scenes.Camera from an engine's camera array."""
    out = []
    for c in arr:
        out.append(scenes.Camera(c.width, c.height, c.fx, c.fy, c.cx, c.cy, np.array(list(c.R)).reshape(3, 3),
                                 np.array(list(c.t)), c.znear))
    return out


def _exact_trim(case, s):
    leaves = [t.detach() for t in _leaves64(s["params"])]
    c = torch.zeros(case["views"], 1, case["n"], device=DEV, dtype=torch.float64)
    for v, arr in enumerate(s["cams"]):
        cam = _cameras(arr)[0]
        with torch.no_grad():
            view = _View(leaves, case["degree"], cam)
            tot = torch.zeros(len(view.ids), device=DEV, dtype=torch.float64)
            cnt = torch.zeros_like(tot)
            for _, px, py in _chunks(cam, view.chunk):
                _, alpha, front, _, _ = view.pixels(px, py)
                on = alpha > 0
                tot += torch.where(on, alpha ** case["gamma"] * front ** (1 - case["gamma"]), 0 * alpha).sum(0)
                cnt += on.sum(0)
            c[v, 0, view.ids] = torch.where(cnt > 0, tot / cnt.clamp(min=1), 0 * tot)
    c_avg = c.sum((0, 1)) / case["views"]
    bound = torch.sort(c_avg).values[int(float(np.float32(case["ratio"])) * (case["n"] - 1))]
    return dict(c_view=c, c_avg=c_avg, bound=bound[None], mask=None, removed=None)


def _exact_action(case, s):
    p, n = s["params"], case["n"]
    ls = p.log_scale.double()
    remove = s["remove"].bool() | (torch.sigmoid(p.opacity_logit.double()) < float(np.float32(0.005)))
    cand = ~remove & (s["mask"] & 4).bool()
    clone = cand & (torch.exp(ls).max(0).values <= float(np.float32(s["scale"])))
    split = cand & ~clone
    keep = ~remove & ~split
    new = torch.where(clone, 1, torch.where(split, 2, 0))
    born = torch.repeat_interleave(torch.arange(n, device=DEV), new)
    child = torch.arange(len(born), device=DEV) - torch.repeat_interleave(torch.cumsum(new, 0) - new, new)
    src = torch.cat([keep.nonzero().reshape(-1), born])
    is_split = torch.cat([torch.zeros(int(keep.sum()), device=DEV, dtype=torch.bool), split[born]])
    which = torch.cat([torch.zeros(int(keep.sum()), device=DEV, dtype=torch.int64), child])
    R = _rotation(p.quat.double())
    z = s["z"].double()[src, which]
    off = sum(torch.exp(ls[k, src]) * z[:, k] * R[:, k, src] for k in (0, 1))
    mean = p.mean.double()[:, src] + torch.where(is_split, off, 0 * off)
    scales = ls[:, src] - torch.where(is_split, math.log(float(np.float32(1.6))), 0.0)
    fresh = torch.arange(len(src), device=DEV) >= int(keep.sum())
    moments = [[torch.where(fresh.view(-1, *([1] * (t.dim() - 1))) if k == 4 else fresh, 0.0,
                            t.double()[src] if k >= 3 else t.double()[:, src]) for k, t in enumerate(m)]
               for m in s["moments"]]
    return dict(actions=None, counts=None, src=None, moments=moments,
                out=[mean, scales, p.quat.double()[:, src], p.opacity_logit.double()[src], p.sh.double()[src]])


def _exact_loss(case, s):
    loss, d, ds = _loss64(s["img"], s["target"])
    return dict(loss=loss, d_img=d, d_img_ssim=ds)


def _exact_crop(case, s):
    pts = s["points"].double()
    count = torch.zeros(pts.shape[1], device=DEV, dtype=torch.int64)
    rho, rf = float(np.float32(s["radius"])), float(np.float32(2.1213))
    for cam in s["cams"]:
        a = cam.as_array()
        W, H, fx, fy, cx, cy = a[:6]
        X = torch.tensor(a[6:15].reshape(3, 3), device=DEV) @ pts + torch.tensor(a[15:18], device=DEV)[:, None]
        Z = X[2]
        seen = torch.ones_like(Z, dtype=torch.bool)
        den = (Z * Z - rho * rho).clamp(min=1e-300)
        for k, (f, c, size) in enumerate(((fx, cx, W), (fy, cy, H))):
            root = rho * torch.sqrt((X[k] ** 2 + Z * Z - rho * rho).clamp(min=0))
            centre = f * X[k] / Z + c
            lo = torch.minimum(f * (X[k] * Z - root) / den + c, centre - rf)
            hi = torch.maximum(f * (X[k] * Z + root) / den + c, centre + rf)
            seen &= torch.ceil(lo - 0.5).clamp(min=0) <= torch.floor(hi - 0.5).clamp(max=size - 1)
        count += (Z > a[18]) & (seen | (Z <= rho))
    T = torch.tensor(s["T"], device=DEV)
    g = T[:, :3] @ pts[:, count >= case["tau"]] + T[:, 3:]
    s["outline"][:, :g.shape[1]] = g[:2]
    return dict(count=None, keep=None, ground=s["outline"], low=float(g[2].min()), high=float(g[2].max()))


def _exact_lloyd(case, s):
    x, cb = s["x"][s["rows"].long()].double(), s["start"].double()
    code = torch.empty(len(x), device=DEV, dtype=torch.int64)
    norm = (cb * cb).sum(1)
    for a in range(0, len(x), 20_000):
        code[a:a + 20_000] = (norm - 2 * x[a:a + 20_000] @ cb.T).argmin(1)
    sums = torch.zeros_like(cb).index_add_(0, code, x)
    cnt = torch.bincount(code, minlength=len(cb))
    return dict(code=None, codebook=torch.where(cnt[:, None] > 0, sums / cnt.clamp(min=1)[:, None], cb), counts=None)
