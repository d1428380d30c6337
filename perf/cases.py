"""Performance cases of the training framework, over the range it is used in.

A case is a dict of plain values with a ``kind``:

* ``step``     one training step of a partition (``train.PlainTrainer``), resumed in
               mid-training with its optimiser moments;
* ``batched``  one step of several uneven partitions and views at once, replayed from its
               captured graph (``train.BatchedTrainer``);
* ``grad``     rendering and loss through autograd, forward and backward, as a program with
               its own optimiser calls them (``ops.render``, ``ops.LossFn``);
* ``view``     one evaluation: a view rendered without per-pixel state and its masked PSNR;
* ``loss``     the masked L1 + D-SSIM loss and its image gradient;
* ``learned``  the learned initialisation of a partition's points (16-NN, features, network);
* ``plain``    the plain k-NN initialisation;
* ``network``  one training step of the initialisation network;
* ``density``  one clone / split / prune pass of the adaptive density control.

``listed()`` names twelve of them, ``draw()`` gives more of the same ranges, ``prepare()`` makes
the inputs on the GPU from a seed, ``run()`` is one pass and ``exact()`` the same values in
64 bits by plain torch.
"""
import math

import numpy as np
import torch

from paper_2509_12138_amd import learned_init, ops, scene, train

DEVICE = "cuda"
SQRT_PI = math.sqrt(math.pi)
NAMES = ops.PARAM_NAMES
LAM = 0.2
STEPS_DONE = 500            # optimiser steps behind a resumed trainer
# Learning rates of the fine-tuning phase (a fiftieth of the defaults): repeated passes then
# stay on about the same Gaussians.
LRS = {k: v * 0.02 for k, v in train.DEFAULT_LR.items()}
EXTENT = 2.75
# (pixel, Gaussian) pairs up to which exact() renders by evaluating every pair
DENSE_PAIRS = 3e9
DENSE_POINTS = 40_000       # points up to which exact() finds neighbours by brute force

# Rasteriser plans in use: an untuned trainer's default, the plan tuned for full-HD views
# (also with reproducible gradient sums), the one tuned for high-resolution views of dense
# partitions, and the memory-saving mode that keeps no per-pixel state.
PLANS = {
    "default": dict(tile=16, schedule="default", chunk=0, waves=1, fixed_sums=False, stored=True),
    "tuned": dict(tile=16, schedule="lpt", chunk=64, waves=4, fixed_sums=False, stored=True),
    "reproducible": dict(tile=16, schedule="lpt", chunk=64, waves=4, fixed_sums=True, stored=True),
    "dense": dict(tile=8, schedule="lpt+split", chunk=128, waves=1, fixed_sums=False, stored=True),
    "recompute": dict(tile=16, schedule="lpt", chunk=0, waves=1, fixed_sums=False, stored=False),
}


def listed():
    return [
        # smoke-sized partition (64^3 field, 4,096 points, 128x128 views): launches and host
        # latency, the untuned trainer
        dict(name="step_small", kind="step", shape="sphere", n=4096, width=128, height=128,
             view=3, plan="default", sh=0, sparse=False),
        # the bench's workload: one million Gaussians, full-HD views, tuned plan
        dict(name="step_1080p", kind="step", shape="layer", n=1_000_000, width=1920, height=1080,
             view=11, plan="tuned", sh=0, sparse=False),
        # one eighth of a hundred-million-Gaussian scene at 3840x2160, tuned plan
        dict(name="step_4k", kind="step", shape="octant", n=13_300_000, width=3840, height=2160,
             view=7, plan="dense", sh=0, sparse=False),
        # view-dependent colour, reproducible sums, ragged sizes
        dict(name="step_sh3", kind="step", shape="layer", n=250_003, width=1237, height=701,
             view=21, plan="reproducible", sh=3, sparse=False),
        # eight uneven partitions, four views each, one graph replay
        dict(name="batched_8x4", kind="batched", shape="sphere", n=800_000, parts=8, views=4,
             width=640, height=360),
        # autograd with default buffers, ragged sizes
        dict(name="grad_ragged", kind="grad", shape="sphere", n=20_011, width=333, height=251,
             view=5, plan="default"),
        # one evaluation view of a trained partition
        dict(name="view_1080p", kind="view", shape="layer", n=1_000_000, width=1920, height=1080,
             view=30, tile=16),
        # the loss of four views
        dict(name="loss_4views", kind="loss", views=4, width=1277, height=717),
        # initialisation of a four-million-point partition by the network
        dict(name="learned_4m", kind="learned", shape="sphere", n=4_000_000),
        # plain initialisation of a mid-sized one
        dict(name="plain_300k", kind="plain", shape="layer", n=300_007),
        # one mini-batch of the network's training at the trainer's default size
        dict(name="network_65k", kind="network", n=262_144, batch=65_536),
        # density control of half a million Gaussians
        dict(name="density_500k", kind="density", n=500_009),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step"] * 6 + ["grad", "grad", "batched", "batched", "view", "loss",
                                      "learned", "plain", "network", "density"])
    width = _log(rng, 96, 2048)
    height = max(48, int(width * rng.uniform(0.5, 1.0)))
    per_pixel = math.exp(rng.uniform(math.log(0.05), math.log(1.2)))
    n = max(1000, min(int(per_pixel * width * height), 2_000_000))
    shape = rng.choice(["sphere", "layer", "octant"])
    view = rng.randrange(64)
    if kind == "step":
        return dict(kind=kind, shape=shape, n=n, width=width, height=height, view=view,
                    plan=rng.choice(sorted(PLANS)), sh=rng.choice([0, 0, 1, 2, 3]),
                    sparse=rng.random() < 0.3)
    if kind == "grad":
        return dict(kind=kind, shape=shape, n=n, width=width, height=height, view=view,
                    plan=rng.choice(sorted(PLANS)))
    if kind == "batched":
        w = _log(rng, 96, 800)
        return dict(kind=kind, shape="sphere", n=_log(rng, 8000, 800_000), parts=rng.randint(2, 8),
                    views=rng.choice([1, 2, 4]), width=w, height=max(48, int(w * 0.6)))
    if kind == "view":
        return dict(kind=kind, shape=shape, n=n, width=width, height=height, view=view,
                    tile=rng.choice([8, 16]))
    if kind == "loss":
        return dict(kind=kind, views=rng.randint(1, 4), width=width, height=height)
    if kind in ("learned", "plain"):
        return dict(kind=kind, shape=shape, n=_log(rng, 2000, 4_000_000))
    if kind == "network":
        batch = _log(rng, 1000, 200_000)
        return dict(kind=kind, n=4 * batch + rng.randrange(1000), batch=batch)
    return dict(kind=kind, n=_log(rng, 2000, 2_000_000))


# --------------------------------------------------------------------------
# Inputs
# --------------------------------------------------------------------------

def _generator(seed):
    return torch.Generator(device=DEVICE).manual_seed(int(seed) * 7919 + 13)


def _rand(gen, *shape):
    return torch.rand(shape, generator=gen, device=DEVICE)


def _randn(gen, *shape):
    return torch.randn(shape, generator=gen, device=DEVICE)


def _morton(p, bits=10):
    """Permutation that sorts points [3, n] along a Z-order curve."""
    lo = p.min(1, keepdim=True).values
    hi = p.max(1, keepdim=True).values
    q = ((p - lo) / (hi - lo).clamp_min(1e-20) * (2 ** bits - 1) + 0.5).to(torch.int64)
    code = torch.zeros_like(q[0])
    for b in range(bits):
        for a in range(3):
            code |= ((q[a] >> b) & 1) << (3 * b + 2 - a)
    return torch.sort(code, stable=True).indices


def _surface(shape, n, gen):
    """n points [3, n] in Z order on an isosurface, their unit normals [3, n] and the mean
    spacing of the samples.  sphere: the bumpy sphere |x| = 0.5 - 0.05 sin 6x sin 6y sin 6z;
    octant: its x, y, z >= 0 part; layer: a mixing layer z = sum of seeded sine modes."""
    if shape == "layer":
        m = scene.MixingInterface(seed=2)
        xy = _rand(gen, 2, n) * 2 - 1
        z, gx, gy = torch.zeros(n, device=DEVICE), 0.0, 0.0
        for (kx, ky), amp, phi in zip(m.k, m.A, m.phi):
            ph = math.pi * (float(kx) * xy[0] + float(ky) * xy[1]) + float(phi)
            z += float(amp) * torch.sin(ph)
            c = (math.pi * float(amp)) * torch.cos(ph)
            gx, gy = gx - float(kx) * c, gy - float(ky) * c
        p = torch.stack([xy[0], xy[1], z])
        nrm = torch.stack([gx, gy, torch.ones_like(z)])
        area = 5.2
    else:
        d = _randn(gen, 3, n)
        d = d / d.norm(dim=0, keepdim=True).clamp_min(1e-6)
        if shape == "octant":
            d = d.abs()
        r = torch.full((n,), 0.5, device=DEVICE)
        for _ in range(12):
            s = torch.sin(6 * r * d)
            r = 0.5 - 0.05 * s[0] * s[1] * s[2]
        p = r * d
        s, c = torch.sin(6 * p), torch.cos(6 * p)
        nrm = d + 0.3 * torch.stack([c[0] * s[1] * s[2], s[0] * c[1] * s[2], s[0] * s[1] * c[2]])
        area = math.pi if shape == "sphere" else math.pi / 8
    nrm = nrm / nrm.norm(dim=0, keepdim=True)
    order = _morton(p)
    return p[:, order].contiguous(), nrm[:, order].contiguous(), math.sqrt(area / n)


def _gaussians(shape, n, gen, sh=0):
    """Gaussians of a partition in mid-training: anisotropic, rotated, varied opacity."""
    p, nrm, spacing = _surface(shape, n, gen)
    quat = 0.3 * _randn(gen, 4, n)
    quat[0] += 1.0
    color = SQRT_PI * nrm + 0.1 * _randn(gen, 3, n)
    if sh:
        color = torch.cat([color, 0.05 * _randn(gen, 3 * (sh + 1) ** 2 - 3, n)])
    return dict(mean=p, log_scale=math.log(0.73 * spacing) + 0.25 * _randn(gen, 3, n),
                quat=quat, opacity_logit=1.2 * _randn(gen, n) - 1.0, color=color.contiguous())


def _cameras(case):
    w, h = case["width"], case["height"]
    orbit = scene.orbit_cameras(64, w, h)
    return orbit[[(case.get("view", 9) + 17 * j) % 64 for j in range(case.get("views", 2))]]


def _targets(params, cams, gen):
    """Target images [V, 3, H, W] and masks [V, H, W] of a partition: its coloured points on a
    coarse grid of cells, smoothed, with a little noise; the mask is the cells they cover."""
    w, h = int(cams[0]["width"]), int(cams[0]["height"])
    cell = 8
    cw, ch = -(-w // cell), -(-h // cell)
    rgb = (0.28209479 * params["color"][:3] + 0.5).clamp(0, 1)
    imgs, masks = [], []
    for cam in cams:
        R = torch.as_tensor(np.array(cam["R"]).reshape(3, 3), device=DEVICE)
        t = torch.as_tensor(np.array(cam["t"]), device=DEVICE)
        x, y, z = [(R[i, :, None] * params["mean"]).sum(0) + t[i] for i in range(3)]
        u = ((float(cam["fx"]) * x / z + float(cam["cx"])) / cell).long()
        v = ((float(cam["fy"]) * y / z + float(cam["cy"])) / cell).long()
        ok = (u >= 0) & (u < cw) & (v >= 0) & (v < ch) & (z > 0.2)
        at = torch.where(ok, v * cw + u, torch.full_like(u, ch * cw))
        grid = torch.full((3, ch * cw + 1), -1.0, device=DEVICE)
        grid = grid.scatter_reduce(1, at.expand(3, -1), rgb, "amax")[:, :-1].reshape(1, 3, ch, cw)
        grid = torch.nn.functional.max_pool2d(grid, 3, 1, 1)
        hit = (grid[0, 0] >= 0).to(torch.uint8)
        img = torch.nn.functional.interpolate(grid.clamp_min(0), scale_factor=cell, mode="bilinear")
        imgs.append(img[0, :, :h, :w])
        masks.append(hit.repeat_interleave(cell, 0).repeat_interleave(cell, 1)[:h, :w])
    img = torch.stack(imgs)
    img = (img + 0.02 * _randn(gen, *img.shape)).clamp(0, 1).contiguous()
    return img, torch.stack(masks).contiguous()


def _moments(params, pixels, gen):
    """Adam moments of a trainer in mid-training: gradients of a loss averaged over pixels."""
    size = dict(mean=50.0, log_scale=0.5, quat=0.2, opacity_logit=0.5, color=1.0)
    m, v = {}, {}
    for k in NAMES:
        s = size[k] / pixels * torch.exp(0.5 * _randn(gen, *params[k].shape))
        m[k] = 0.3 * s * _randn(gen, *params[k].shape)
        v[k] = s * s
    return m, v


def _step_inputs(case, seed):
    gen = _generator(seed)
    params = _gaussians(case["shape"], case["n"], gen, case.get("sh", 0))
    cams = _cameras(case)
    targets, masks = _targets(params, cams, gen)
    m, v = _moments(params, case["width"] * case["height"], gen)
    return params, cams, targets, masks, m, v


def _resume(trainer, m, v, adam):
    """Puts a checkpoint's moments and step count into a new trainer."""
    for k in NAMES:
        trainer.m[k].copy_(m[k])
        trainer.v[k].copy_(v[k])
    adam.step_dev.fill_(STEPS_DONE)


def _image(shape, gen):
    """Smooth images [S, 3, H, W] with values in about [0.1, 0.9]."""
    S, H, W = shape
    small = _rand(gen, S, 3, max(2, H // 16), max(2, W // 16))
    img = torch.nn.functional.interpolate(small, size=(H, W), mode="bilinear")
    return (0.1 + 0.8 * img).contiguous()


def _loss_inputs(case, seed):
    gen = _generator(seed)
    S, H, W = case["views"], case["height"], case["width"]
    target = _image((S, H, W), gen)
    image = (target + 0.03 * _randn(gen, S, 3, H, W)).clamp_min(0).contiguous()
    y = torch.arange(H, device=DEVICE)[:, None] / H - 0.5
    x = torch.arange(W, device=DEVICE)[None, :] / W - 0.5
    wob = 0.05 * torch.sin(9 * torch.atan2(y, x) + seed % 7)
    mask = ((x * x + y * y).sqrt() < 0.42 + wob).to(torch.uint8)     # a silhouette
    return image, target, mask.expand(S, H, W).contiguous()


def _network_inputs(case, seed):
    gen = _generator(seed)
    x = (0.5 * _randn(gen, case["n"], 96)).to(torch.bfloat16)
    t = torch.cat([0.4 * _randn(gen, case["n"], 3) - 0.3,
                   torch.nn.functional.normalize(_randn(gen, case["n"], 4), dim=1),
                   _randn(gen, case["n"], 1)], 1).contiguous()
    w = learned_init.InitMLP.random(seed=seed % 1000, device=DEVICE).w
    m, v = {}, {}
    for k in learned_init.MLP_NAMES:
        s = 1e-2 * torch.exp(0.3 * _randn(gen, *w[k].shape))
        m[k], v[k] = 0.1 * s * _randn(gen, *w[k].shape), s * s
    return x, t, w, m, v


def _density_inputs(case, seed):
    """Gaussians with the statistics of a hundred steps: a twentieth is faint, three in a hundred
    small ones and three in a hundred large ones have a screen-space gradient above the threshold."""
    gen = _generator(seed)
    n = case["n"]
    params = _gaussians("layer", n, gen)
    m, v = _moments(params, 1e6, gen)
    th = _density_thresholds(case)
    who = torch.randperm(n, generator=gen, device=DEVICE)
    faint, small, large = (who[int(a * n):int(b * n)]
                           for a, b in ((0, 0.05), (0.05, 0.08), (0.08, 0.11)))
    params["opacity_logit"].clamp_(min=th["min_opacity_logit"] + 0.1)
    params["opacity_logit"][faint] = th["min_opacity_logit"] - 0.5
    cut = th["max_log_scale_clone"]
    params["log_scale"][:, small] = params["log_scale"][:, small].clamp(max=cut - 0.01)
    params["log_scale"][0, large] = cut + 0.05 + 0.3 * _rand(gen, len(large))
    denom = 1 + torch.floor(99 * _rand(gen, n))
    mean = th["grad_threshold"] * (0.1 + 0.8 * _rand(gen, n))
    for grow in (small, large):
        mean[grow] = th["grad_threshold"] * (1.1 + 2 * _rand(gen, len(grow)))
    return params, m, v, (denom * mean).contiguous(), denom, _randn(gen, n, 2, 3)


def _density_thresholds(case):
    spacing = math.sqrt(5.2 / case["n"])
    return dict(grad_threshold=2e-4, max_log_scale_clone=math.log(spacing),
                min_opacity_logit=math.log(0.02 / 0.98), max_log_scale=float("inf"),
                log_split=math.log(1.6))


# --------------------------------------------------------------------------
# prepare and run
# --------------------------------------------------------------------------

def prepare(case, seed):
    kind = case["kind"]
    s = dict(kind=kind)
    if kind == "step":
        params, cams, targets, masks, m, v = _step_inputs(case, seed)
        pl = PLANS[case["plan"]]
        tr = train.PlainTrainer(
            params, cams, targets, masks, tile=(pl["tile"], pl["tile"]), lam=LAM,
            stored=pl["stored"], extent=EXTENT, lrs=LRS, schedule=pl["schedule"],
            chunk=pl["chunk"], fwd_waves=pl["waves"], deterministic=pl["fixed_sums"],
            sh_degree=case["sh"], sh_up_every=0, sparse_adam=case["sparse"], device=DEVICE)
        tr.fit_capacity()
        _resume(tr, m, v, tr.dev_adam)
        s["trainer"] = tr
    elif kind == "batched":
        gen = _generator(seed)
        cams = _cameras(case)
        share = np.arange(1, case["parts"] + 1, dtype=np.float64)
        counts = np.maximum(200, case["n"] * share / share.sum()).astype(int)
        whole = _gaussians(case["shape"], int(counts.sum()), gen)
        by_x = torch.sort(whole["mean"][0]).indices       # slabs along x
        m, v = _moments(whole, case["width"] * case["height"], gen)
        parts, at = [], 0
        for c in counts:
            idx = torch.sort(by_x[at:at + int(c)]).values
            at += int(c)
            part = {k: whole[k][..., idx].contiguous() for k in NAMES}
            targets, masks = _targets(part, cams, gen)
            parts.append(dict(params={k: t.cpu().numpy() for k, t in part.items()},
                              targets=targets, masks=masks))
        tr = train.BatchedTrainer(parts, cams, views_per_part=case["views"], lrs=LRS,
                                  extent=EXTENT, device=DEVICE)
        tr.fit_capacity()
        tr.prepare()
        _resume(tr, m, v, tr.adam)
        s["trainer"] = tr
    elif kind == "grad":
        params, cams, targets, masks, _, _ = _step_inputs(case, seed)
        pl = PLANS[case["plan"]]
        views = ops.Views.single(case["n"], cams[:1], DEVICE)
        bufs = ops.RasterBuffers(views, case["width"], case["height"], (pl["tile"], pl["tile"]),
                                 store_state=pl["stored"])
        bufs.set_schedule(pl["schedule"], chunk=pl["chunk"], fwd_waves=pl["waves"],
                          deterministic=pl["fixed_sums"])
        s.update(params={k: t.clone().requires_grad_() for k, t in params.items()}, bufs=bufs,
                 target=targets[:1].contiguous(), mask=masks[:1].contiguous(),
                 loss=ops.LossBuffers(1, case["height"], case["width"], DEVICE))
    elif kind == "view":
        params, cams, targets, masks, _, _ = _step_inputs(case, seed)
        views = ops.Views.single(case["n"], cams[:1], DEVICE)
        bufs = ops.RasterBuffers(views, case["width"], case["height"],
                                 (case["tile"], case["tile"]), store_state=False)
        s.update(params=params, bufs=bufs, target=targets[:1].contiguous(),
                 mask=masks[:1].contiguous(),
                 psnr=ops.PsnrBuffers(1, case["height"], case["width"], DEVICE))
    elif kind == "loss":
        image, target, mask = _loss_inputs(case, seed)
        s.update(image=image, target=target, mask=mask,
                 loss=ops.LossBuffers(case["views"], case["height"], case["width"], DEVICE))
    elif kind in ("learned", "plain"):
        gen = _generator(seed)
        s["points"], s["normals"], _ = _surface(case["shape"], case["n"], gen)
        if kind == "learned":
            s["mlp"] = learned_init.InitMLP.random(seed=seed % 1000, device=DEVICE)
    elif kind == "network":
        x, t, w, m, v = _network_inputs(case, seed)
        tr = learned_init.MLPTrainer(learned_init.InitMLP(w), x.view(torch.int16), t,
                                     lr=2e-5, batch=case["batch"], seed=seed % 1000)
        for k in learned_init.MLP_NAMES:
            tr.m[k].copy_(m[k])
            tr.v[k].copy_(v[k])
        tr.steps = STEPS_DONE
        s["trainer"] = tr
    else:
        params, m, v, accum, denom, z = _density_inputs(case, seed)
        d = ops.Densifier(case["n"], DEVICE)
        d.accum.copy_(accum)
        d.denom.copy_(denom)
        s.update(params=params, m=m, v=v, z=z, densifier=d, thresholds=_density_thresholds(case))
    return s


def run(s):
    kind = s["kind"]
    if kind == "step":
        tr = s["trainer"]
        tr.step(tr.step_count % tr.V)
        return dict(params=tr.params, m=tr.m, v=tr.v, loss=tr.loss.loss, image=tr.bufs.image)
    if kind == "batched":
        tr = s["trainer"]
        tr.step(0)
        return dict(params=tr.params, m=tr.m, v=tr.v, loss=tr.loss.loss, image=tr.bufs.image)
    if kind == "grad":
        for t in s["params"].values():
            t.grad = None
        image = ops.render(s["params"], s["bufs"])
        loss = ops.LossFn.apply(image, s["target"], s["mask"], LAM, s["loss"])
        loss.sum().backward()
        return dict(image=image, loss=loss, grads={k: t.grad for k, t in s["params"].items()})
    if kind == "view":
        s["bufs"].render_checked(ops.gaussians_struct(s["params"]))
        psnr = s["psnr"](s["bufs"].image, s["target"], s["mask"])
        return dict(image=s["bufs"].image, psnr=psnr)
    if kind == "loss":
        loss, d_image = s["loss"](s["image"], s["target"], s["mask"], LAM, 1.0)
        return dict(loss=loss, d_image=d_image)
    if kind == "learned":
        return learned_init.learned_params(s["mlp"], s["points"], s["normals"])
    if kind == "plain":
        return learned_init.plain_init(s["points"], s["normals"])
    if kind == "network":
        tr = s["trainer"]
        loss = tr.step()
        return dict(loss=loss, weights=tr.mlp.w, m=tr.m, v=tr.v)
    d, th = s["densifier"], s["thresholds"]
    n_out = d.select(s["params"], s["m"], s["v"], **th)
    P, M, V = d.apply(s["params"], s["m"], s["v"], n_out, s["z"], th["log_split"])
    return dict(n=n_out, params=P, m=M, v=V, action=d.action)


# --------------------------------------------------------------------------
# What a pass cannot do without
# --------------------------------------------------------------------------

BLENDS_PER_PIXEL = 40       # entries a foreground pixel blends (measured at 1080p)


def work(case):
    kind = case["kind"]
    n = case.get("n", 0)
    px = case.get("width", 0) * case.get("height", 0)
    rows = 11 + 3 * (case.get("sh", 0) + 1) ** 2
    blends = BLENDS_PER_PIXEL * px * 0.65
    if kind == "step":        # parameters and moments in and out, target and mask in
        return dict(bytes=24 * rows * n + 13 * px, flops=72 * blends + 700 * px + 300 * n)
    if kind == "batched":
        v = case["views"] * case["parts"]
        return dict(bytes=24 * rows * n + 13 * px * v,
                    flops=72 * blends * v / case["parts"] + 700 * px * v
                    + 300 * n * case["views"])
    if kind == "grad":        # parameters in, gradients and image out
        return dict(bytes=8 * rows * n + 25 * px, flops=72 * blends + 700 * px + 300 * n)
    if kind == "view":
        return dict(bytes=4 * rows * n + 25 * px, flops=22 * blends + 20 * px + 150 * n)
    if kind == "loss":
        return dict(bytes=37 * px * case["views"], flops=700 * px * case["views"])
    if kind == "learned":     # points and normals in, 14 parameters out
        return dict(bytes=80 * n, flops=(21504 + 16 * 60) * n)
    if kind == "plain":
        return dict(bytes=80 * n, flops=60 * n)
    if kind == "network":
        return dict(bytes=(192 + 32) * case["batch"], flops=4 * 21504 * case["batch"])
    return dict(bytes=(2 * 3 * 4 * 14 + 12 + 24) * n, flops=30 * n)


# --------------------------------------------------------------------------
# The same values in 64 bits
# --------------------------------------------------------------------------

def _f64(d):
    return {k: t.detach().double() for k, t in d.items()}


def _sh_basis(d, degree):
    """Real spherical harmonics (Condon-Shortley phase) of unit directions [3, n]."""
    x, y, z = d
    pi = math.pi
    Y = [torch.full_like(x, 0.5 / math.sqrt(pi))]
    if degree > 0:
        c = math.sqrt(3 / (4 * pi))
        Y += [-c * y, c * z, -c * x]
    if degree > 1:
        c = 0.5 * math.sqrt(15 / pi)
        Y += [c * x * y, -c * y * z, 0.25 * math.sqrt(5 / pi) * (3 * z * z - 1), -c * x * z,
              0.5 * c * (x * x - y * y)]
    if degree > 2:
        a, b = 0.25 * math.sqrt(35 / (2 * pi)), 0.5 * math.sqrt(105 / pi)
        e = 0.25 * math.sqrt(21 / (2 * pi))
        Y += [-a * y * (3 * x * x - y * y), b * x * y * z, -e * y * (5 * z * z - 1),
              0.25 * math.sqrt(7 / pi) * z * (5 * z * z - 3), -e * x * (5 * z * z - 1),
              0.5 * b * z * (x * x - y * y), -a * x * (x * x - 3 * y * y)]
    return Y


def _project64(p, cam):
    """Projected Gaussians [9, n] (mean, conic, opacity, colour), depth and visibility."""
    R = torch.as_tensor(np.array(cam["R"], np.float64).reshape(3, 3), device=DEVICE)
    t = torch.as_tensor(np.array(cam["t"], np.float64), device=DEVICE)
    fx, fy, cx, cy = (float(cam[k]) for k in ("fx", "fy", "cx", "cy"))
    W, H = int(cam["width"]), int(cam["height"])
    x, y, z = [sum(R[i, j] * p["mean"][j] for j in range(3)) + t[i] for i in range(3)]
    q = p["quat"] / p["quat"].norm(dim=0, keepdim=True)
    w, a, b, c = q
    rot = [[1 - 2 * (b * b + c * c), 2 * (a * b - w * c), 2 * (a * c + w * b)],
           [2 * (a * b + w * c), 1 - 2 * (a * a + c * c), 2 * (b * c - w * a)],
           [2 * (a * c - w * b), 2 * (b * c + w * a), 1 - 2 * (a * a + b * b)]]
    s = torch.exp(p["log_scale"])
    # J R: the two image rows of the perspective map's Jacobian, in world axes
    lx, ly = 1.3 * W / (2 * fx), 1.3 * H / (2 * fy)
    ux, uy = (x / z).clamp(-lx, lx), (y / z).clamp(-ly, ly)
    rows = []
    for f, u, r in ((fx, ux, 0), (fy, uy, 1)):
        g = [f / z * (R[r, j] - u * R[2, j]) for j in range(3)]
        rows.append([s[k] * sum(g[j] * rot[j][k] for j in range(3)) for k in range(3)])
    c11 = sum(v * v for v in rows[0]) + 0.3
    c12 = sum(u * v for u, v in zip(*rows))
    c22 = sum(v * v for v in rows[1]) + 0.3
    det = c11 * c22 - c12 * c12
    o = torch.sigmoid(p["opacity_logit"])
    centre = -(R.T @ t)
    d = p["mean"] - centre[:, None]
    d = d / d.norm(dim=0, keepdim=True)
    degree = int(round(math.sqrt(p["color"].shape[0] / 3))) - 1
    basis = _sh_basis(d, degree)
    rgb = [torch.relu(sum(Y * p["color"][3 * k + ch] for k, Y in enumerate(basis)) + 0.5)
           for ch in range(3)]
    rec = torch.stack([fx * x / z + cx, fy * y / z + cy, c22 / det, -c12 / det, c11 / det, o]
                      + rgb)
    return rec, z.detach(), (z.detach() > float(cam["znear"])) & (255 * o.detach() > 1)


def _composite64(rec, px, py):
    """Colour [P, 3] of the pixels with centres (px, py) over depth-ordered Gaussians."""
    dx, dy = px[:, None] - rec[0], py[:, None] - rec[1]
    power = -0.5 * (rec[2] * dx * dx + rec[4] * dy * dy) - rec[3] * dx * dy
    raw = rec[5] * torch.exp(power)
    alpha = torch.where(raw < 0.99, raw, torch.full_like(raw, 0.99))
    alpha = torch.where((power <= 0) & (alpha >= 1 / 255), alpha, torch.zeros_like(alpha))
    own = torch.log1p(-alpha)
    total = torch.cumsum(own, 1)
    weight = alpha * torch.exp(total - own) * (total.detach() >= math.log(1e-4))
    return torch.stack([(weight * rec[6 + c]).sum(1) for c in range(3)], 1)


def _pixel_chunks(n, W, H):
    step = max(1, int(1.5e7 // max(n, 1)))
    i = torch.arange(W * H, device=DEVICE)
    for lo in range(0, W * H, step):
        at = i[lo:lo + step]
        yield at, (at % W).double() + 0.5, (at // W).double() + 0.5


def _render64(params, cam):
    """Image [3, H, W] and the function that takes its gradient to the parameters'."""
    W, H = int(cam["width"]), int(cam["height"])
    leaf = {k: t.clone().requires_grad_() for k, t in params.items()}
    rec, depth, seen = _project64(leaf, cam)
    order = torch.sort(torch.where(seen, depth, torch.full_like(depth, math.inf)),
                       stable=True).indices[:int(seen.sum())]
    held = rec[:, order].detach()
    image = torch.zeros(W * H, 3, dtype=torch.float64, device=DEVICE)
    with torch.no_grad():
        for at, px, py in _pixel_chunks(len(order), W, H):
            image[at] = _composite64(held, px, py)

    def backward(d_image):
        d = d_image.reshape(3, -1).T
        held.requires_grad_()
        for at, px, py in _pixel_chunks(len(order), W, H):
            if bool((d[at] != 0).any()):
                (_composite64(held, px, py) * d[at]).sum().backward()
        rec[:, order].backward(held.grad if held.grad is not None else torch.zeros_like(held))
        return {k: t.grad if t.grad is not None else torch.zeros_like(t) for k, t in leaf.items()}

    return image.T.reshape(3, H, W), backward


def _blur64(a):
    w = [math.exp(-(i - 5) ** 2 / (2 * 1.5 ** 2)) for i in range(11)]
    H, W = a.shape[-2:]
    for dim, size in ((-1, W), (-2, H)):
        pad = torch.nn.functional.pad(a, (5, 5, 0, 0) if dim == -1 else (0, 0, 5, 5))
        a = sum(w[i] / sum(w) * pad.narrow(dim, i, size) for i in range(11))
    return a


def _loss64(image, target, mask):
    """Loss of one image [3, H, W] and its gradient."""
    img = image.detach().clone().requires_grad_()
    m = mask.double()
    x, y = m * img, m * target.double()
    mx, my = _blur64(x), _blur64(y)
    vx, vy, cov = _blur64(x * x) - mx * mx, _blur64(y * y) - my * my, _blur64(x * y) - mx * my
    ssim = ((2 * mx * my + 1e-4) * (2 * cov + 9e-4)
            / ((mx * mx + my * my + 1e-4) * (vx + vy + 9e-4)))
    loss = (1 - LAM) * (x - y).abs().mean() + LAM * (1 - ssim.mean())
    loss.backward()
    return loss.detach(), img.grad


def _adam64(p, g, m, v, lr, b1, b2, eps, t):
    m2 = {k: b1 * m[k].double() + (1 - b1) * g[k] for k in p}
    v2 = {k: b2 * v[k].double() + (1 - b2) * g[k] ** 2 for k in p}
    new = {k: p[k] - lr[k] * (m2[k] / (1 - b1 ** t)) / ((v2[k] / (1 - b2 ** t)).sqrt() + eps)
           for k in p}
    return new, m2, v2


def _neighbours64(points, k):
    """Indices and distances [n, k] of the k nearest other points, by brute force."""
    p = points.double()
    n = p.shape[1]
    idx, dist = [], []
    for lo in range(0, n, 2048):
        q = p[:, lo:lo + 2048]
        d2 = sum((q[a][:, None] - p[a][None, :]) ** 2 for a in range(3))
        r = torch.arange(q.shape[1], device=DEVICE)
        d2[r, lo + r] = math.inf
        v, i = torch.topk(d2, k, dim=1, largest=False)
        idx.append(i)
        dist.append(v.sqrt())
    return torch.cat(idx), torch.cat(dist)


def _network64(w, x):
    w = _f64(w)
    h = torch.relu(x @ w["w1"] + w["b1"])
    return torch.relu(h @ w["w2"] + w["b2"]) @ w["w3"] + w["b3"]


def _quat_of(F):
    """Unit quaternions [4, n] of rotation matrices given as rows of [n] tensors."""
    (a, b, c), (d, e, f), (g, h, i) = F
    cand = torch.stack([torch.stack([1 + a + e + i, h - f, c - g, d - b]),
                        torch.stack([h - f, 1 + a - e - i, b + d, c + g]),
                        torch.stack([c - g, b + d, 1 - a + e - i, f + h]),
                        torch.stack([d - b, c + g, f + h, 1 - a - e + i])])
    best = torch.stack([cand[k, k] for k in range(4)]).argmax(0)
    q = cand.gather(0, best.expand(1, 4, -1))[0]
    return q / q.norm(dim=0, keepdim=True)


def _learned64(mlp, points, normals):
    p, nrm = points.double(), normals.double()
    n = p.shape[1]
    idx, dist = _neighbours64(points, 16)
    dbar = dist.mean(1)
    z = nrm / nrm.norm(dim=0, keepdim=True)
    e = torch.nn.functional.one_hot(z.abs().argmin(0), 3).T.double()
    x = torch.linalg.cross(z, e, dim=0)
    x = x / x.norm(dim=0, keepdim=True)
    y = torch.linalg.cross(z, x, dim=0)
    feats = []
    for k in range(16):
        j = idx[:, k]
        for v in ((p[:, j] - p) / dbar, nrm[:, j]):
            feats += [(ax * v).sum(0) for ax in (x, y, z)]
    out = _network64(mlp.w, torch.stack(feats, 1))
    qf = _quat_of([[x[i], y[i], z[i]] for i in range(3)])          # local -> world
    ql = (out[:, 3:7] / out[:, 3:7].norm(dim=1, keepdim=True)).T
    w0, a0, b0, c0 = qf
    w1, a1, b1, c1 = ql
    q = torch.stack([w0 * w1 - a0 * a1 - b0 * b1 - c0 * c1, w0 * a1 + a0 * w1 + b0 * c1 - c0 * b1,
                     w0 * b1 - a0 * c1 + b0 * w1 + c0 * a1, w0 * c1 + a0 * b1 - b0 * a1 + c0 * w1])
    q = torch.where(q[0] < 0, -q, q)
    return dict(mean=p, log_scale=torch.log(dbar) + out[:, :3].T, quat=q, opacity_logit=out[:, 7],
                color=SQRT_PI * nrm)


def _network_step64(case, seed):
    x, t, w, m, v = _network_inputs(case, seed)
    perm = torch.randperm(case["n"], generator=torch.Generator(device="cpu").manual_seed(seed % 1000))
    rows = perm[:min(case["batch"], case["n"])].to(DEVICE)
    leaf = {k: a.detach().double().clone().requires_grad_() for k, a in w.items()}
    h = torch.relu(x[rows].double() @ leaf["w1"] + leaf["b1"])
    y = torch.relu(h @ leaf["w2"] + leaf["b2"]) @ leaf["w3"] + leaf["b3"]
    tt = t[rows].double()
    sq = ((y[:, :3] - tt[:, :3]) ** 2).sum(1) + (y[:, 7] - tt[:, 7]) ** 2
    dot = ((y[:, 3:7] / y[:, 3:7].norm(dim=1, keepdim=True)) * tt[:, 3:7]).sum(1)
    loss = (sq + 1 - dot.abs()).mean()
    loss.backward()
    p = {k: a.detach() for k, a in leaf.items()}
    g = {k: a.grad for k, a in leaf.items()}
    new, m2, v2 = _adam64(p, g, m, v, {k: 2e-5 for k in p}, 0.9, 0.999, 1e-8, STEPS_DONE + 1)
    return dict(loss=loss.detach().reshape(1), weights=new, m=m2, v=v2)


def _density64(case, seed):
    params, m, v, accum, denom, z = _density_inputs(case, seed)
    th = {k: torch.tensor(x, dtype=torch.float32, device=DEVICE)
          for k, x in _density_thresholds(case).items()}
    top = params["log_scale"].max(0).values
    grow = (denom > 0) & (accum.double() >= th["grad_threshold"].double() * denom.double())
    small = top <= th["max_log_scale_clone"]
    action = torch.where(grow, torch.where(small, 2, 3), 1)
    action = torch.where(params["opacity_logit"] < th["min_opacity_logit"], 0, action)
    outs = torch.tensor([0, 1, 2, 2], device=DEVICE)[action]
    src = torch.repeat_interleave(torch.arange(case["n"], device=DEVICE), outs)
    first = torch.cumsum(outs, 0) - outs
    child = torch.arange(len(src), device=DEVICE) - first[src]
    split = action[src] == 3
    P = {k: t.double()[..., src] for k, t in params.items()}
    q = P["quat"] / P["quat"].norm(dim=0, keepdim=True)
    w, a, b, c = q
    e = torch.exp(P["log_scale"]) * z.double()[src, child].T
    off = torch.stack([
        (1 - 2 * (b * b + c * c)) * e[0] + 2 * (a * b - w * c) * e[1] + 2 * (a * c + w * b) * e[2],
        2 * (a * b + w * c) * e[0] + (1 - 2 * (a * a + c * c)) * e[1] + 2 * (b * c - w * a) * e[2],
        2 * (a * c - w * b) * e[0] + 2 * (b * c + w * a) * e[1] + (1 - 2 * (a * a + b * b)) * e[2]])
    P["mean"] = torch.where(split, P["mean"] + off, P["mean"])
    P["log_scale"] = torch.where(split, P["log_scale"] - math.log(1.6), P["log_scale"])
    fresh = split | (child == 1)                 # children and copies start without moments
    M, V = ({k: torch.where(fresh, torch.zeros((), dtype=torch.float64, device=DEVICE),
                            t.double()[..., src]) for k, t in d.items()} for d in (m, v))
    return dict(n=None, params=P, m=M, v=V, action=None)


def exact(case, seed):
    kind = case["kind"]
    pairs = case.get("n", 0) * case.get("width", 0) * case.get("height", 0)
    if kind in ("step", "grad", "view") and pairs <= DENSE_PAIRS:
        params, cams, targets, masks, m, v = _step_inputs(case, seed)
        image, backward = _render64(_f64(params), cams[0])
        if kind == "view":
            mk = masks[0].double()
            se = (mk * (image.clamp(0, 1) - targets[0].double()) ** 2).sum()
            psnr = 10 * torch.log10(3 * mk.sum() / se)
            return dict(image=image[None], psnr=psnr.reshape(1))
        loss, d_image = _loss64(image, targets[0], masks[0])
        grads = backward(d_image)
        if kind == "grad":
            return dict(image=image[None], loss=loss.reshape(1), grads=grads)
        t = STEPS_DONE + 1
        lr0, lr1 = LRS["mean"] * EXTENT, 1.6e-6 * EXTENT
        lr = dict(LRS, mean=lr0 * (lr1 / lr0) ** (t / 30000.0))
        rows = torch.full((params["color"].shape[0], 1), LRS["color_rest"], dtype=torch.float64,
                          device=DEVICE)
        rows[:3] = LRS["color"]
        lr["color"] = rows
        p = _f64(params)
        new, m2, v2 = _adam64(p, grads, m, v, lr, 0.9, 0.999, 1e-15, t)
        if case["sparse"]:
            return dict(loss=loss.reshape(1), image=image[None])
        return dict(params=new, m=m2, v=v2, loss=loss.reshape(1), image=image[None])
    if kind == "loss":
        image, target, mask = _loss_inputs(case, seed)
        got = [_loss64(image[i].double(), target[i], mask[i]) for i in range(case["views"])]
        return dict(loss=torch.stack([g[0] for g in got]), d_image=torch.stack([g[1] for g in got]))
    if kind in ("learned", "plain") and case["n"] <= DENSE_POINTS:
        points, normals, _ = _surface(case["shape"], case["n"], _generator(seed))
        if kind == "learned":
            mlp = learned_init.InitMLP.random(seed=seed % 1000, device=DEVICE)
            return _learned64(mlp, points, normals)
        d = _neighbours64(points, 3)[1].mean(1).clamp_min(1e-6)
        n = case["n"]
        one = torch.ones(n, dtype=torch.float64, device=DEVICE)
        op = learned_init.PLAIN_OPACITY
        return dict(mean=points.double(), log_scale=torch.log(d).expand(3, n),
                    quat=torch.stack([one, 0 * one, 0 * one, 0 * one]),
                    opacity_logit=math.log(op / (1 - op)) * one, color=SQRT_PI * normals.double())
    if kind == "network":
        return _network_step64(case, seed)
    if kind == "density":
        return _density64(case, seed)
    return None
