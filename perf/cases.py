"""The work that a user of this framework has it do, as cases that can be measured.

Scenes are drawn with the recipe of ``paper_2510_09997_amd.synth`` (uniform cube or a mixture of
64 clusters, log-scales around exp(-4), SH coefficients of degree 0 to 3, one decay factor per
Gaussian), on the GPU, so that a state of several million Gaussians is made in a moment.  Scenes
that are served are stored as a server stores them (Morton order, a packed copy of the SH
coefficients); scenes that are trained keep the planes only.

Kinds of case
  render    one forward pass of a batch of views: an interactive frame, the LoD frames of one
            pose, a serving batch of mixed sizes, a distant or a budgeted view, strips of a frame
  count     the kept and rendered counts of many views without rendering
  train     forward, loss and backward of one or several views (single step or trainer)
  autograd  the differentiable render inside a PyTorch graph, forward and backward
  loss      the rendering loss and its gradient (L1, or L1 and D-SSIM)
  adam      the fused optimiser step over every parameter plane
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2510_09997_amd import render as R
from paper_2510_09997_amd import synth
from paper_2510_09997_amd.train import DEFAULT_LRS, FusedAdam, MultiViewTrainer

PLANES = ("mean", "log_scale", "quat", "opacity", "decay", "sh")
DEVICE = "cuda"


def _case(kind, name=None, **kw):
    c = dict(kind=kind, n=10000, degree=3, layout="mixture", served=False, poses=1, levels=1, width=256, height=256,
             mixed=False, near=3.0, far=30.0, sv_max=16.0, budget=0, strips=0, waits=False, dssim=0.0)
    c.update(kw)
    if name is not None:
        c["name"] = name
    return c


def listed():
    return [
        # The smallest call: one view of a small object, as in an editor or a test; the time is
        # launches and their latency.
        _case("render", "view_256_10k", n=10_000, degree=0, layout="uniform", width=256, height=256, near=2.5, far=3.5,
              sv_max=1.0, waits=True),
        # An interactive viewer: one frame of a served scene, waiting for its pair count.
        _case("render", "view_1080p_3m", n=3_000_000, served=True, width=1920, height=1080, waits=True),
        # The LoD frames (s_v = 1, 2, 4, 8, 16) of one pose in one pass: the headline benchmark.
        _case("render", "lod5_1080p_3m", n=3_000_000, served=True, levels=5, width=1920, height=1080),
        # A serving batch: six requests of different poses, sizes (720p, 1080p, 4K) and scales.
        _case("render", "serve_mixed_3m", n=3_000_000, served=True, poses=6, width=1920, height=1080, mixed=True),
        # A distant view of a large scene: a few tiles hold very long lists.
        _case("render", "far_1080p_6m", n=6_000_000, served=True, width=1920, height=1080, near=70.0, far=110.0),
        # A frame under a primitive budget, as four strips with their own virtual distance.
        _case("render", "budget_strips_3m", n=3_000_000, served=True, width=1920, height=1080, near=6.0, far=12.0,
              budget=400_000, strips=4),
        # Kept ratios over a sweep of 64 distances without rendering, as a scheduler of detail asks.
        _case("count", "count_64_views_6m", n=6_000_000, served=True, poses=64, width=1920, height=1080, near=2.0,
              far=200.0),
        # One training iteration on one image (forward, L1 and point-count loss, backward).
        _case("train", "train_1view_1m", n=1_000_000, width=1297, height=840, near=4.0, far=6.0, sv_max=8.0, waits=True),
        # The batched training step: sixteen images of three sizes, with the D-SSIM term.
        _case("train", "train_16view_2m", n=2_000_000, poses=16, width=1297, height=840, mixed=True, near=4.0, far=6.0,
              sv_max=8.0, dssim=0.2),
        # The render as a node of a PyTorch graph, two small views of odd size.
        _case("autograd", "autograd_20k", n=20_011, degree=2, poses=2, width=333, height=217, near=4.0, far=6.0, sv_max=4.0),
        # The rendering loss of a batch of two images with its gradient.
        _case("loss", "loss_dssim_1080p", n=20_000, degree=0, poses=2, width=1920, height=1080, near=4.0, far=6.0,
              sv_max=4.0, dssim=0.2),
        # The optimiser step over a scene.
        _case("adam", "adam_2m", n=2_000_000),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["render", "render", "render", "render", "train", "train", "count", "autograd", "loss", "adam"])
    degree = rng.choice([0, 1, 2, 3, 3])
    width, height = _log_int(rng, 200, 1920), _log_int(rng, 130, 1080)
    near = math.exp(rng.uniform(math.log(2.5), math.log(20.0)))
    views = dict(degree=degree, layout=rng.choice(["mixture", "mixture", "uniform"]), width=width, height=height,
                 near=near, far=near * rng.uniform(1.0, 3.0), sv_max=rng.choice([1.0, 4.0, 8.0, 16.0]))
    if kind == "render":
        style = rng.choice(["view", "levels", "serve", "far", "budget", "strips"])
        c = _case("render", **views, n=_log_int(rng, 10_000, 3_000_000), served=rng.random() < 0.7,
                  waits=rng.random() < 0.5)
        if style == "levels":
            c["levels"] = rng.randint(2, 5)
        elif style == "serve":
            c.update(poses=rng.randint(2, 6), mixed=True)
        elif style == "far":
            far = math.exp(rng.uniform(math.log(30.0), math.log(100.0)))
            c.update(near=far, far=far * 1.5, layout="mixture")
        elif style == "budget":
            c["budget"] = max(1, int(c["n"] * rng.uniform(0.02, 0.6)))
        elif style == "strips":
            c["strips"] = rng.randint(2, 5)
        return c
    if kind == "train":
        poses = rng.choice([1, 1, 2, 5, 9])
        return _case("train", **views, n=_log_int(rng, 10_000, 1_500_000), poses=poses, mixed=poses > 1 and rng.random() < 0.5,
                     dssim=rng.choice([0.0, 0.2]), waits=rng.random() < 0.3)
    if kind == "count":
        return _case("count", **views, n=_log_int(rng, 10_000, 6_000_000), poses=rng.randint(1, 64),
                     served=rng.random() < 0.5)
    if kind == "autograd":
        return _case("autograd", **views, n=_log_int(rng, 5_000, 300_000), poses=rng.randint(1, 3))
    if kind == "loss":
        return _case("loss", **views, n=_log_int(rng, 5_000, 50_000), poses=rng.randint(1, 4), dssim=rng.choice([0.0, 0.2, 0.5]))
    return _case("adam", degree=degree, n=_log_int(rng, 10_000, 2_000_000))


# ---------------------------------------------------------------------------------- inputs

def _generator(seed, salt):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(1_000_003 * int(seed) + salt)
    return g


def _planes(case, seed):
    n, K = case["n"], (case["degree"] + 1) ** 2
    g = _generator(seed, 1)
    normal = lambda *s: torch.randn(*s, generator=g, device=DEVICE)
    unit = lambda *s: torch.rand(*s, generator=g, device=DEVICE)
    if case["layout"] == "uniform":
        mean = 2.0 * unit(3, n) - 1.0
    else:
        centres = 10.0 * unit(3, 64) - 5.0
        pick = torch.randint(0, 64, (n,), generator=g, device=DEVICE)
        mean = (centres[:, pick] + 0.3 * normal(3, n)).clamp_(-5.0, 5.0)
    quat = normal(4, n)
    quat /= quat.norm(dim=0, keepdim=True).clamp_min(1e-12)
    sh = normal(K, 3, n)
    sh[0] *= synth.DC_STD
    sh[1:] *= synth.HIGHER_SH_STD
    return dict(n=n, sh_degree=case["degree"], mean=mean, log_scale=-4.0 + 0.5 * normal(3, n), quat=quat,
                opacity=normal(n), decay=0.5 * normal(n), sh=sh.contiguous())


def _views(case, seed):
    rng = np.random.default_rng(1_000_003 * int(seed) + 2)
    poses = case["poses"]
    dirs = synth.unit_vectors(rng, poses)
    radii = np.exp(rng.uniform(math.log(case["near"]), math.log(case["far"]), poses))
    if case["kind"] == "count":
        radii = case["near"] * (case["far"] / case["near"]) ** (np.arange(poses) / max(1, poses - 1))
    svs = np.exp(rng.uniform(0.0, math.log(case["sv_max"]), poses))
    w, h = case["width"], case["height"]
    sizes = [(w, h)]
    if case["mixed"]:
        # 1080p with 720p and 4K beside it; training images in half and one and a half sizes.
        sizes = [(w * 2 // 3, h * 2 // 3), (w, h), (2 * w, 2 * h)] if case["kind"] == "render" else \
                [(w // 2, h // 2), (w, h), (w * 3 // 2, h * 3 // 2)]
    out = []
    for j in range(poses):
        vw, vh = sizes[j % len(sizes)]
        levels = [2.0 ** k for k in range(case["levels"])] if case["levels"] > 1 else [svs[j]]
        for s in levels:
            v = synth.look_at(dirs[j] * radii[j], width=vw, height=vh, s_v=float(s))
            v.budget = case["budget"]
            out += synth.strips(v, [float(2 ** k) for k in range(case["strips"])]) if case["strips"] else [v]
    return out


def _uniform(seed, salt, *shape):
    return torch.rand(*shape, generator=_generator(seed, salt), device=DEVICE)


def _scene(case, seed):
    return R.Scene(_planes(case, seed), packed_sh=case["served"], spatial_order=case["served"])


def _sized_batch(scene, views):
    """A batch whose pair buffer fits the views, as a program that knows its scene keeps it."""
    b = R.Batch(scene.n, views)
    b.project(scene)
    pairs = b.bin_sort()
    del b
    b = R.Batch(scene.n, views, dup_capacity=int(pairs * 1.25) + 65536)
    b.project(scene)
    b.bin_sort(sync=False)
    return b


def _adam_state(case, seed):
    """Parameters, gradients and moments in the middle of a training run."""
    g = _generator(seed, 3)
    planes = _planes(case, seed)
    grads = {k: 1e-4 * torch.randn(planes[k].shape, generator=g, device=DEVICE) for k in PLANES}
    m = {k: 1e-4 * torch.randn(planes[k].shape, generator=g, device=DEVICE) for k in PLANES}
    v = {k: 1e-8 * torch.rand(planes[k].shape, generator=g, device=DEVICE) for k in PLANES}
    return planes, grads, m, v


ADAM_STEPS_DONE = 99


def prepare(case, seed):
    kind = case["kind"]
    if kind == "adam":
        planes, grads, m, v = _adam_state(case, seed)
        scene = R.Scene(planes)
        opt = FusedAdam(scene)
        for k in PLANES:
            opt.m[k].copy_(m[k])
            opt.v[k].copy_(v[k])
        opt.t = ADAM_STEPS_DONE
        return dict(kind=kind, scene=scene, opt=opt, grads=grads)
    scene, views = _scene(case, seed), _views(case, seed)
    s = dict(kind=kind, scene=scene, views=views, waits=case["waits"], sv_max=case["sv_max"], dssim=case["dssim"])
    if kind == "count":
        s["batch"] = R.Batch(scene.n, views, dup_capacity=1)
    elif kind == "train" and (case["poses"] > 1 or case["dssim"] > 0):
        s["trainer"] = MultiViewTrainer(scene, views, s_max=case["sv_max"], lambda_dssim=case["dssim"])
        s["trainer"].set_target(_uniform(seed, 4, 3 * s["trainer"].batch.pixels))
    else:
        s["batch"] = b = _sized_batch(scene, views)
        if kind == "train":
            s["target"] = _uniform(seed, 4, 3 * b.pixels)
            s["grads"] = scene.zeros_like()
        elif kind == "loss":
            # The rendered image close to its target, as in training.
            s["target"] = _uniform(seed, 4, 3 * b.pixels)
            s["rgb"] = (s["target"] + 0.1 * (_uniform(seed, 5, 3 * b.pixels) - 0.5)).clamp_(0.0, 1.0)
        elif kind == "autograd":
            s["leaves"] = [scene.t[k].clone().requires_grad_(True) for k in PLANES]
            s["g_rgb"] = _uniform(seed, 6, 3 * b.pixels) - 0.5
            s["g_eta"] = _uniform(seed, 7, len(views))
    return s


def run(s):
    kind = s["kind"]
    if kind == "render":
        if s["waits"]:
            rgb, T, last, _ = R.render(s["scene"], s["views"], batch=s["batch"])
            return dict(rgb=rgb, T=T, last=last)
        b = s["batch"]
        b.project(s["scene"])
        b.bin_sort(sync=False)
        rgb, T, last = b.render_fwd()
        return dict(rgb=rgb, T=T, last=last)
    if kind == "count":
        return s["batch"].lod_count(s["scene"])
    if kind == "train":
        if "trainer" in s:
            t = s["trainer"]
            t.step()
            return dict(loss=t.loss, grads=t.grads, rgb=t.rgb)
        loss, grads, rgb = R.train_step(s["scene"], s["batch"], s["target"], s["sv_max"], grads=s["grads"],
                                        sync_sort=s["waits"])
        return dict(loss=loss, grads=grads, rgb=rgb)
    if kind == "autograd":
        rgb, eta, T, last = R.ClodRender.apply(*s["leaves"], s["batch"], s["scene"].sh_degree)
        grads = torch.autograd.grad([rgb, eta], s["leaves"], [s["g_rgb"], s["g_eta"]])
        return dict(rgb=rgb, eta=eta, T=T, last=last, grads=list(grads))
    if kind == "loss":
        loss, dL_drgb, dL_deta = s["batch"].loss(s["rgb"], s["target"], s["sv_max"], lambda_dssim=s["dssim"])
        return dict(loss=loss, dL_drgb=dL_drgb, dL_deta=dL_deta)
    opt = s["opt"]
    opt.step(s["grads"], DEFAULT_LRS)
    return dict(param=dict(s["scene"].t), m=opt.m, v=opt.v)


def work(case):
    """Bytes: what every pass reads (means, opacity and decay of every Gaussian; image, target or
    gradient where there is one) and writes (images, gradients).  Which Gaussians are rendered,
    and so how much of the rest is read, depends on the drawn scene and is left out.  Flops: the
    distance, frustum test and Eq. (2) of every (view, Gaussian), the loss's windows, Adam."""
    n, params = case["n"], case["n"] * (12 + 3 * (case["degree"] + 1) ** 2)
    if case["kind"] == "adam":
        return dict(bytes=28 * params, flops=14 * params)
    views = _views(case, 0)
    px = sum(v.width * v.height for v in views)
    project = 60 * n * len(views)
    windows = (2 * (5 + 3) * 22 * 3 + 120) * px
    if case["kind"] == "render":
        return dict(bytes=20 * n + 20 * px, flops=project)
    if case["kind"] == "count":
        return dict(bytes=20 * n + 24 * len(views), flops=project)
    if case["kind"] == "loss":
        return dict(bytes=36 * px, flops=(windows if case["dssim"] > 0 else 6 * px))
    grads = 4 * params
    if case["kind"] == "autograd":
        return dict(bytes=20 * n + 20 * px + 12 * px + grads, flops=3 * project)
    return dict(bytes=20 * n + 24 * px + grads, flops=3 * project + (windows if case["dssim"] > 0 else 6 * px))


# ---------------------------------------------------------------------------------- 64-bit values

def exact(case, seed):
    kind = case["kind"]
    if kind == "adam":
        return _exact_adam(case, seed)
    if kind == "loss":
        return _exact_loss(case, seed)
    pixels = sum(v.width * v.height for v in _views(case, seed)) if kind in ("autograd", "render") else 0
    if kind == "autograd" and case["n"] <= 60_000 and pixels <= 400_000:
        return _exact_render(case, seed, True)
    if (kind == "render" and case["n"] <= 60_000 and pixels <= 400_000 and not case["served"] and not case["strips"]
            and not case["budget"]):
        return _exact_render(case, seed, False)
    return None


def _exact_adam(case, seed):
    planes, grads, m, v = _adam_state(case, seed)
    b1, b2, eps, t = (float(np.float32(x)) for x in (0.9, 0.999, 1e-15, ADAM_STEPS_DONE + 1))
    out = dict(param={}, m={}, v={})
    for k in PLANES:
        p, g = planes[k].double(), grads[k].double()
        m1 = b1 * m[k].double() + (1 - b1) * g
        v1 = b2 * v[k].double() + (1 - b2) * g * g
        step = (m1 / (1 - b1 ** t)) / ((v1 / (1 - b2 ** t)).sqrt() + eps)
        if k == "sh":
            step[0] *= float(np.float32(DEFAULT_LRS["sh_dc"]))
            step[1:] *= float(np.float32(DEFAULT_LRS["sh_rest"]))
        else:
            step *= float(np.float32(DEFAULT_LRS[k]))
        out["param"][k], out["m"][k], out["v"][k] = p - step, m1, v1
    return out


def _exact_loss(case, seed):
    views = _views(case, seed)
    px = sum(v.width * v.height for v in views)
    target = _uniform(seed, 4, 3 * px)
    rgb = (target + 0.1 * (_uniform(seed, 5, 3 * px) - 0.5)).clamp_(0.0, 1.0)
    lam, s_max = case["dssim"], case["sv_max"]
    x = torch.arange(11, dtype=torch.float64, device=DEVICE) - 5
    g = torch.exp(-x * x / (2 * 1.5 * 1.5))
    g = g / g.sum()

    def blur(a):
        a = torch.nn.functional.pad(a, (5, 5, 5, 5))
        h, w = a.shape[1] - 10, a.shape[2] - 10
        a = sum(g[k] * a[:, :, k:k + w] for k in range(11))
        return sum(g[k] * a[:, k:k + h] for k in range(11))

    grads, o = [], 0
    for v in views:
        k = 3 * v.width * v.height
        a = rgb[o:o + k].double().view(3, v.height, v.width).requires_grad_(True)
        b = target[o:o + k].double().view(3, v.height, v.width)
        o += k
        l = (1 - lam) * (a - b).abs().mean()
        if lam > 0:
            mx, my = blur(a), blur(b)
            sxx, syy, sxy = blur(a * a) - mx * mx, blur(b * b) - my * my, blur(a * b) - mx * my
            s = (2 * mx * my + 0.01 ** 2) * (2 * sxy + 0.03 ** 2) / ((mx * mx + my * my + 0.01 ** 2) * (sxx + syy + 0.03 ** 2))
            l = l + lam * (1 - s.mean())
        l = (1 - 0.5 * v.s_v / s_max) ** 2 * l
        l.backward()
        grads.append(a.grad.reshape(-1))
    # The point-count term depends on the counts of the projection: no value here.
    return dict(loss=None, dL_drgb=torch.cat(grads), dL_deta=None)


def _exact_render(case, seed, backward):
    """A splatting renderer in 64 bits, tile by tile, with its gradients."""
    planes, views = _planes(case, seed), _views(case, seed)
    n = case["n"]
    leaves = [planes[k].double().requires_grad_(backward) for k in PLANES]
    mean, log_scale, quat, opacity, decay, sh = leaves
    px = sum(v.width * v.height for v in views)
    g_rgb, g_eta = _uniform(seed, 6, 3 * px) - 0.5, _uniform(seed, 7, len(views))
    f64 = lambda a: torch.as_tensor(np.asarray(a), dtype=torch.float64, device=DEVICE)
    total, rgbs, Ts, etas, base = 0.0, [], [], [], 0
    tau, eps, near_z, guard, dilation = (float(np.float32(x)) for x in (1.0 / 255.0, 1e-6, 0.2, 1.3, 0.3))
    for vi, v in enumerate(views):
        W, t, c = f64(v.W), f64(v.t), f64(v.c)
        x, y, z = W @ mean + t[:, None]
        frustum = (z > near_z) & (x.abs() <= guard * 0.5 * v.width / v.fx * z) & (y.abs() <= guard * 0.5 * v.height / v.fy * z)
        e = mean - c[:, None]
        d = e.square().sum(0).sqrt()
        d_max = d[frustum].max() if bool(frustum.any()) else torch.ones((), dtype=torch.float64, device=DEVICE)
        q = (d / d_max * v.s_v) ** 2 / (2 * decay.clamp_min(0) ** 2 + eps)
        a2 = torch.sigmoid(opacity) * torch.exp(-q)
        kept = a2 > tau * v.s_v
        etas.append(kept.double().mean())
        qn = quat / quat.norm(dim=0, keepdim=True)
        w_, x_, y_, z_ = qn
        Rm = torch.stack([1 - 2 * (y_ * y_ + z_ * z_), 2 * (x_ * y_ - w_ * z_), 2 * (x_ * z_ + w_ * y_),
                          2 * (x_ * y_ + w_ * z_), 1 - 2 * (x_ * x_ + z_ * z_), 2 * (y_ * z_ - w_ * x_),
                          2 * (x_ * z_ - w_ * y_), 2 * (y_ * z_ + w_ * x_), 1 - 2 * (x_ * x_ + y_ * y_)]).view(3, 3, n)
        M = (Rm * torch.exp(log_scale)[None]).permute(2, 0, 1)
        S = (M.unsqueeze(2) * M.unsqueeze(1)).sum(3)
        zero = torch.zeros_like(z)
        J = torch.stack([v.fx / z, zero, -v.fx * x / z ** 2, zero, v.fy / z, -v.fy * y / z ** 2]).view(2, 3, n).permute(2, 0, 1)
        T2 = (J.unsqueeze(3) * W.view(1, 1, 3, 3)).sum(2)
        U = (T2.unsqueeze(3) * S.unsqueeze(1)).sum(2)
        ca, cb, cc = (U[:, 0] * T2[:, 0]).sum(1) + dilation, (U[:, 0] * T2[:, 1]).sum(1), (U[:, 1] * T2[:, 1]).sum(1) + dilation
        det = ca * cc - cb * cb
        mid = 0.5 * (ca + cc)
        rad = torch.ceil(3 * (mid + (mid * mid - det).clamp_min(0).sqrt()).sqrt()).detach()
        u, w = v.fx * x / z + v.cx, v.fy * y / z + v.cy
        tw, th = (v.width + 15) // 16, (v.height + 15) // 16
        x0, x1 = torch.floor((u - rad) / 16).clamp(0, tw), (torch.floor((u + rad) / 16) + 1).clamp(0, tw)
        y0, y1 = torch.floor((w - rad) / 16).clamp(0, th), (torch.floor((w + rad) / 16) + 1).clamp(0, th)
        drawn = frustum & kept & (det > 0) & (x0 < x1) & (y0 < y1)
        order = torch.nonzero(drawn).squeeze(1)
        order = order[torch.argsort(z[order].detach(), stable=True)]
        D = e / d
        colour = ((sh * _sh_basis(case["degree"], D)[:, None]).sum(0) + 0.5).clamp_min(0)
        screen = torch.stack([u, w, cc / det, -cb / det, ca / det, a2, colour[0], colour[1], colour[2]])[:, order]
        box = torch.stack([x0, x1, y0, y1])[:, order].detach()
        leaf = screen.detach().requires_grad_(backward)
        rgb = torch.zeros(3, v.height, v.width, dtype=torch.float64, device=DEVICE)
        Tm = torch.ones(v.height, v.width, dtype=torch.float64, device=DEVICE)
        gi = g_rgb[3 * base:3 * (base + v.width * v.height)].double().view(3, v.height, v.width)
        base += v.width * v.height
        for ty in range(th):
            row = torch.nonzero((box[2] <= ty) & (box[3] > ty)).squeeze(1)
            if not len(row):
                continue
            for tx in range(tw):
                at = row[(box[0, row] <= tx) & (box[1, row] > tx)]
                if not len(at):
                    continue
                g = leaf[:, at]
                py, pxs = torch.meshgrid(torch.arange(16 * ty, min(16 * ty + 16, v.height), device=DEVICE),
                                         torch.arange(16 * tx, min(16 * tx + 16, v.width), device=DEVICE), indexing="ij")
                py, pxs = py.reshape(-1), pxs.reshape(-1)
                dx, dy = g[0][:, None] - (pxs + 0.5), g[1][:, None] - (py + 0.5)
                power = -0.5 * (g[2][:, None] * dx * dx + g[4][:, None] * dy * dy) - g[3][:, None] * dx * dy
                alpha = (g[5][:, None] * torch.exp(power)).clamp_max(0.99)
                used = (power <= 0) & (alpha >= float(np.float32(1 / 255)))
                alpha = torch.where(used, alpha, torch.zeros_like(alpha))
                after = torch.cumprod(1 - alpha.detach(), 0)
                alpha = torch.where(after >= float(np.float32(1e-4)), alpha, torch.zeros_like(alpha))
                after = torch.cumprod(1 - alpha, 0)
                before = torch.cat([torch.ones_like(after[:1]), after[:-1]])
                out = g[6:9] @ (alpha * before)
                rgb[:, py, pxs], Tm[py, pxs] = out.detach(), after[-1].detach()
                if backward:
                    total_tile = (out * gi[:, py, pxs]).sum()
                    total_tile.backward()
        if backward:
            total = total + (screen * leaf.grad).sum() + g_eta[vi].double() * a2.mean()
        rgbs.append(rgb)
        Ts.append(Tm)
    if not backward:
        if case["waits"]:
            return dict(rgb=rgbs, T=Ts, last=[None] * len(views))
        return dict(rgb=torch.cat([a.reshape(-1) for a in rgbs]), T=torch.cat([a.reshape(-1) for a in Ts]), last=None)
    grads = torch.autograd.grad(total, leaves, allow_unused=True)
    grads = [torch.zeros_like(p) if g is None else g for g, p in zip(grads, leaves)]
    return dict(rgb=torch.cat([a.reshape(-1) for a in rgbs]), eta=torch.stack(etas),
                T=torch.cat([a.reshape(-1) for a in Ts]), last=None, grads=grads)


def _sh_basis(degree, D):
    """Real spherical harmonics of unit directions D [3][n], order l = 0 .. degree, m = -l .. l."""
    X, Y, Z = D
    pi = math.pi
    out = [torch.full_like(X, 0.5 / math.sqrt(pi))]
    if degree > 0:
        k = math.sqrt(3 / (4 * pi))
        out += [k * Y, k * Z, k * X]
    if degree > 1:
        a, b, c = math.sqrt(15 / pi) / 2, math.sqrt(5 / pi) / 4, math.sqrt(15 / pi) / 4
        out += [a * X * Y, a * Y * Z, b * (2 * Z * Z - X * X - Y * Y), a * X * Z, c * (X * X - Y * Y)]
    if degree > 2:
        a, b, c = math.sqrt(35 / (2 * pi)) / 4, math.sqrt(105 / pi) / 2, math.sqrt(21 / (2 * pi)) / 4
        e, f = math.sqrt(7 / pi) / 4, math.sqrt(105 / pi) / 4
        out += [a * Y * (3 * X * X - Y * Y), b * X * Y * Z, c * Y * (4 * Z * Z - X * X - Y * Y),
                e * Z * (2 * Z * Z - 3 * X * X - 3 * Y * Y), c * X * (4 * Z * Z - X * X - Y * Y),
                f * Z * (X * X - Y * Y), a * X * (X * X - 3 * Y * Y)]
    return torch.stack(out)
