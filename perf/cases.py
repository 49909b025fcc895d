"""What users of this renderer have it do, as measurable cases.

``listed()`` names one case per kind of use at the sizes of this repository's
workloads, tests and benchmark; ``draw()`` gives more of the same kinds over
the ranges between them. Every case goes through the public Python entry
points (render_forward / render_backward, the autograd render, one training
step, the tabulated schedule, the learned surrogate and its training).
``exact()`` evaluates the same outputs from the paper's formulas in 64 bits
with torch alone.

Kinds:
  frame      forward render with a workspace kept between frames
  step       forward + backward with that workspace (the host sums several
             views' losses itself)
  autograd   the differentiable render without a workspace: every call
             allocates and reads the list count back
  train      one optimisation step of the whole objective (penalty, L1,
             D-SSIM, Adam)
  tabulated  forward render on the per-pixel table, the moment bounds or the
             learned network at its nodes
  surrogate  forward + backward through the per-query network
  fit        one training step of that network on a minibatch
"""
import math
import random
from types import SimpleNamespace

import numpy as np
import torch

import paper_2512_11800_amd as M
from paper_2512_11800_amd import surrogate, train

PARAMS = ("means", "scales", "quats", "densities", "colors")
HIDDEN, INPUTS, NODES = 64, 7, 32


# ---------------------------------------------------------------------------
# The cases
# ---------------------------------------------------------------------------
def _case(kind, n=0, width=0, height=0, **more):
    c = {"kind": kind, "n": n, "width": width, "height": height, "cams": 1, "clusters": 64, "sh": 3,
         "moments": 4, "intervals": 3, "trig": False, "penalty": False, "network": False, "batch": 0}
    c.update(more)
    return c


def listed():
    small = {"clusters": 0, "sh": -1}  # uniform RGB scene, as the small test scenes are
    return [
        # a viewer's thumbnail or a unit test: launches and host latency
        _case("frame", 2000, 128, 128, name="frame_small", **small),
        # fitting a small scene through torch autograd, odd image size
        _case("autograd", 20000, 397, 301, name="autograd_small", penalty=True, **small),
        # an interactive full-HD frame of a trained-size scene
        _case("frame", 500_000, 1920, 1080, name="frame_1080p"),
        # that view forward and backward
        _case("step", 500_000, 1920, 1080, name="step_1080p"),
        # the paper's six moments, forward and backward
        _case("step", 500_000, 1920, 1080, name="step_1080p_k6", moments=6),
        # the finest reconstruction the library has, odd image size
        _case("step", 100_000, 1003, 757, name="step_k8_n5", moments=8, intervals=5),
        # the paper's ablation with trigonometric moments
        _case("step", 200_000, 1280, 720, name="step_trig", trig=True),
        # a training step of the whole objective at the paper's image size
        _case("train", 1_000_000, 1600, 1064, name="train_1m"),
        # a large batched step: several 4K views of a large scene at once
        _case("step", 3_000_000, 3840, 2160, name="batch_4k", cams=4, clusters=256),
        # a full-HD frame with the learned network on the per-pixel table
        _case("tabulated", 500_000, 1920, 1080, name="tabulated_network", moments=6, network=True),
        # forward and backward through the per-query network
        _case("surrogate", 100_000, 960, 540, name="surrogate_step", moments=6),
        # training that network: the minibatch its training loop defaults to
        _case("fit", name="fit_network", batch=65536),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["frame", "frame", "step", "step", "autograd", "train", "tabulated", "surrogate", "fit"])
    if kind == "fit":
        return _case("fit", batch=_log_int(rng, 1000, 262144))
    if kind == "autograd":  # small scenes
        return _case(kind, _log_int(rng, 500, 40000), rng.randint(64, 640), rng.randint(64, 480), clusters=0,
                     sh=-1, moments=rng.choice([4, 6]), intervals=rng.choice([3, 5]),
                     penalty=rng.random() < 0.5)
    width = _log_int(rng, 160, 1920)
    height = max(96, min(1200, int(width * rng.uniform(0.5, 0.8))))
    if kind == "surrogate":
        return _case(kind, _log_int(rng, 5000, 150_000), min(width, 960), min(height, 640), moments=6,
                     intervals=rng.choice([3, 5]))
    c = _case(kind, _log_int(rng, 3000, 1_000_000), width, height, sh=rng.choice([-1, 0, 1, 2, 3, 3]))
    if kind == "tabulated":
        c["network"] = rng.random() < 0.5
        c["moments"] = 6 if c["network"] else rng.choice([4, 6])
    elif kind == "train":
        c["moments"] = rng.choice([4, 4, 6])
    else:
        c["cams"] = rng.choice([1, 1, 1, 2, 3])
        c["moments"] = rng.choice([4, 4, 6, 6, 8])
        c["intervals"] = rng.choice([3, 3, 5])
        c["trig"] = c["moments"] == 4 and rng.random() < 0.15
        c["penalty"] = rng.random() < 0.25
    if c["moments"] == 8:
        c["n"] = min(c["n"], 200_000)
    return c


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------
def _camera(position, width, height, background):
    """60 degree pinhole camera at `position` looking at the origin (OpenCV axes)."""
    p = np.asarray(position, np.float64)
    fwd = -p / np.linalg.norm(p)
    right = np.cross(fwd, (0.0, 1.0, 0.0))
    right /= np.linalg.norm(right)
    r = np.stack([right, np.cross(fwd, right), fwd])
    w2c = np.concatenate([r, (-r @ p)[:, None]], 1).astype(np.float32)
    f = float(np.float32(height / 2.0 / math.tan(math.radians(30.0))))
    return SimpleNamespace(world_to_cam=w2c, fx=f, fy=f, cx=width / 2.0, cy=height / 2.0, width=width,
                           height=height, t_near=float(np.float32(0.2)), background=background)


def _inputs(case, seed):
    """The scene, cameras, options and the gradients or targets of a case, from the seed alone."""
    gen = torch.Generator(device="cuda").manual_seed(seed)

    def normal(*shape):
        return torch.randn(*shape, generator=gen, device="cuda")

    def uniform(*shape):
        return torch.rand(*shape, generator=gen, device="cuda")

    s = SimpleNamespace()
    if case["kind"] in ("surrogate", "fit") or case["network"]:  # He-initialised network, small biases
        s.theta = torch.cat([(normal(HIDDEN, INPUTS) * (2 / INPUTS) ** 0.5).reshape(-1), 0.1 * normal(HIDDEN),
                             (normal(HIDDEN, HIDDEN) * (2 / HIDDEN) ** 0.5).reshape(-1), 0.1 * normal(HIDDEN),
                             normal(HIDDEN) * (1 / HIDDEN) ** 0.5, 0.1 * normal(1)])
    if case["kind"] == "fit":
        b = case["batch"]
        f = normal(b, 8)
        f[:, 0], f[:, 1] = 0.0, math.asinh(1.0)  # standardised mean and variance
        f[:, 3] = torch.asinh(3.0 + 4.0 * f[:, 3].abs())
        f[:, 4] *= 2.0
        f[:, 5] = torch.asinh(15.0 + 60.0 * f[:, 5].abs())
        f[:, 6] = (2.0 * f[:, 6]).clamp(-10, 10)
        f[:, 7] = torch.exp(f[:, 7])
        s.x, s.t = f.contiguous(), torch.exp(-f[:, 7] * uniform(b)).contiguous()
        # the moments of an optimiser in the middle of a run
        s.m, s.v = 1e-3 * normal(s.theta.numel()), 1e-5 * (0.5 + uniform(s.theta.numel()))
        return s
    n, deg = case["n"], case["sh"]
    if case["clusters"]:
        centres = 8.0 * uniform(case["clusters"], 3) - 4.0
        which = torch.randint(0, case["clusters"], (n,), generator=gen, device="cuda")
        means = centres[which] + 0.3 * normal(n, 3)
        scales, densities = torch.exp(-4.0 + 0.7 * normal(n, 3)), torch.exp(1.5 * normal(n))
        distance, background = 10.0, (0.0, 0.0, 0.0)
    else:
        means = 2.0 * uniform(n, 3) - 1.0
        scales, densities = torch.exp(-3.0 + 0.5 * normal(n, 3)), torch.exp(normal(n))
        distance, background = 3.0, (0.25, 0.5, 0.75)
    quats = torch.nn.functional.normalize(normal(n, 4), dim=1)
    colors = uniform(n, 3) if deg < 0 else 0.2 * normal(n, (deg + 1) ** 2, 3)
    s.params = {"means": means, "scales": scales, "quats": quats, "densities": densities, "colors": colors}
    s.params = {k: v.contiguous() for k, v in s.params.items()}
    rng = random.Random(seed)
    s.cams = []
    for i in range(case["cams"]):
        if i == 0:
            p = (0.0, 0.0, -distance)
        else:
            a, h = rng.uniform(0, 2 * math.pi), rng.uniform(-0.8, 0.8)
            r = math.sqrt(1 - h * h)
            p = (distance * r * math.cos(a), distance * h, distance * r * math.sin(a))
        s.cams.append(_camera(p, case["width"], case["height"], background))
    f32 = lambda x: float(np.float32(x))  # noqa: E731
    s.opts = SimpleNamespace(n_moments=case["moments"], n_intervals=case["intervals"], kappa=3.0,
                             conf_c=f32(0.01), beta=0.25, eps=f32(1e-6), full_coverage=False,
                             basis="trigonometric" if case["trig"] else "power")
    c, h, w = case["cams"], case["height"], case["width"]
    if case["kind"] in ("step", "autograd", "surrogate"):
        s.grad_image = normal(c, h, w, 3) / (h * w)
        s.grad_penalty = (0.1 / (c * h * w) * torch.ones(c, h, w, device="cuda")) if case["penalty"] else None
    if case["kind"] == "train":
        low = uniform(1, 3, max(2, h // 16), max(2, w // 16))  # a smooth photograph-like target
        s.target = torch.nn.functional.interpolate(low, (h, w), mode="bilinear")
        s.target = s.target.permute(0, 2, 3, 1).contiguous()
        s.lrs = {"means": 1.6e-4, "scales": 2e-5, "quats": 1e-3, "densities": 5e-3, "colors": 2.5e-3}
        s.m = {k: 1e-9 * normal(*v.shape) for k, v in s.params.items()}
        s.v = {k: 1e-16 * (0.5 + uniform(*v.shape)) for k, v in s.params.items()}
    return s


STEP = 200  # optimiser steps taken before the measured one


def prepare(case, seed):
    s = _inputs(case, seed)
    s.case = case
    if case["kind"] == "fit":
        s.step = STEP
        s.packed = surrogate.mlp_pack(s.theta)
        return s
    s.ws = M.Workspace()
    if case["kind"] == "surrogate" or case["network"]:
        s.packed = surrogate.mlp_pack(s.theta)
    if case["kind"] in ("autograd", "surrogate"):
        for v in s.params.values():
            v.requires_grad_(True)
    else:
        s.g = M.Gaussians(*(s.params[k] for k in PARAMS), case["sh"])
    if case["kind"] == "train":
        s.adam = train.Adam(s.lrs, step=STEP, m=s.m, v=s.v)
    return s


def run(s):
    case = s.case
    kind = case["kind"]
    if kind == "frame":
        out = M.render_forward(s.g, s.cams, s.opts, ws=s.ws, penalty=case["penalty"], on_device=True)
        return {"image": out[0], "penalty": out[3]} if case["penalty"] else {"image": out[0]}
    if kind == "step":
        out = M.render_forward(s.g, s.cams, s.opts, ws=s.ws, penalty=case["penalty"], on_device=True)
        grads = M.render_backward(s.g, s.cams, s.opts, out[2], out[1], s.grad_image, s.grad_penalty)
        return {"image": out[0], "grads": grads}
    if kind == "autograd":
        p = [s.params[k] for k in PARAMS]
        out = M.render(*p, s.cams, s.opts, sh_degree=case["sh"], with_penalty=case["penalty"])
        outs, gos = ([out], [s.grad_image]) if not case["penalty"] else (list(out), [s.grad_image, s.grad_penalty])
        grads = torch.autograd.grad(outs, p, gos)
        return {"image": outs[0], "grads": dict(zip(PARAMS, grads))}
    if kind == "surrogate":
        p = [s.params[k] for k in PARAMS]
        image = M.render_surrogate(*p, s.cams, s.packed, s.opts, sh_degree=case["sh"], ws=s.ws)
        grads = torch.autograd.grad([image], p, [s.grad_image])
        return {"image": image, "grads": dict(zip(PARAMS, grads))}
    if kind == "tabulated":
        out = M.render_forward_tabulated(s.g, s.cams, s.opts, s.packed if case["network"] else None, NODES, ws=s.ws)
        return {"image": out[0]}
    if kind == "train":
        out = train.train_step(s.g, s.cams, s.opts, s.target, s.adam, ws=s.ws, on_device=True)
        return {"params": {k: getattr(s.g, k) for k in PARAMS}, "l1": out["l1"], "dssim": out["dssim"],
                "consistency": out["consistency"], "total": out["total"]}
    loss, grad = surrogate.mlp_loss_grad(s.packed, s.x, s.t)
    s.step += 1
    surrogate.adam_step(s.theta, s.m, s.v, grad, s.step, 1e-3)
    surrogate.mlp_pack(s.theta, s.packed)
    return {"loss": loss, "grad": grad, "theta": s.theta, "m": s.m, "v": s.v}


# ---------------------------------------------------------------------------
# Work
# ---------------------------------------------------------------------------
def _pairs(case):
    """Covering (pixel, Gaussian) pairs to expect: the mean share of the image a Gaussian of the scene covers."""
    return (4.3e-5 if case["clusters"] else 4e-3) * case["n"] * case["cams"] * case["width"] * case["height"]


def work(case):
    """Inputs read and outputs written once; operations counted from the method's formulas per covering pair
    (moments; edges with one reconstruction each; in the backward their adjoints), per network evaluation
    (multiply-adds of the three layers) and per pixel of the losses' windows."""
    macs = HIDDEN * INPUTS + HIDDEN * HIDDEN + HIDDEN
    if case["kind"] == "fit":
        p = macs + 2 * HIDDEN + 1
        return {"bytes": case["batch"] * 36 + p * 28, "flops": 6.0 * macs * case["batch"]}
    n, k, ne = case["n"], case["moments"], case["intervals"] + 1
    per = 11 + (3 if case["sh"] < 0 else 3 * (case["sh"] + 1) ** 2)  # floats per Gaussian
    px = case["cams"] * case["width"] * case["height"]
    pairs = _pairs(case)
    recon, herm = {4: (73, 85), 6: (169, 165), 8: (340, 232)}[k]
    moments = 49 + 18 + 7 * (k - 1) + k + 1
    if case["kind"] == "tabulated":
        nodes = px * NODES * (2.0 * macs if case["network"] else recon)
        return {"bytes": 4.0 * (n * per + 3 * px), "flops": pairs * (moments + 45 + 20 * ne) + nodes}
    quad = 45 + ne * (13 + recon) + 9 * (ne - 1)
    flops = pairs * (moments + quad)
    nbytes = 4.0 * (n * per + 3 * px)
    if case["kind"] == "surrogate":
        flops = pairs * (2 * moments + 400 + ne * 6.0 * macs)
    elif case["kind"] != "frame":
        flops += pairs * (quad + ne * (herm + 4 * k + 20) + 20 * (ne - 1) + 90 + 159 + 3 * moments)
    if case["kind"] != "frame":
        nbytes += 4.0 * (n * per + 3 * px)  # gradients out, the image's gradient in
    if case["kind"] == "train":
        nbytes += 4.0 * (n * per * 6 + 6 * px)  # Adam's moments and parameters, the target
        flops += px * 3 * 400.0
    return {"bytes": nbytes, "flops": flops}


# ---------------------------------------------------------------------------
# The same outputs in 64 bits, from the paper's formulas (no kernel of this
# repository): Gaussians to ray-space coefficients and screen rectangles, all
# covering (pixel, Gaussian) pairs of a block of image rows at a time, torch
# autograd for the gradients.
# ---------------------------------------------------------------------------
MIX = (1e-3, 1e-2, 1e-1, 1.0)  # mixture weights of the degenerate-measure rule
SPAN = 1.8 * math.pi           # arc of the circle the depths fill


def _sh_basis(d, degree):
    x, y, z = d.unbind(-1)
    out = [torch.full_like(x, math.sqrt(1 / (4 * math.pi)))]
    if degree > 0:
        c = math.sqrt(3 / (4 * math.pi))
        out += [c * y, c * z, c * x]
    if degree > 1:
        c = math.sqrt(15 / math.pi) / 2
        out += [c * x * y, c * y * z, math.sqrt(5 / math.pi) / 4 * (3 * z * z - 1), c * x * z, c / 2 * (x * x - y * y)]
    if degree > 2:
        a, b = math.sqrt(35 / (2 * math.pi)) / 4, math.sqrt(105 / math.pi) / 2
        e, f = math.sqrt(21 / (2 * math.pi)) / 4, math.sqrt(7 / math.pi) / 4
        out += [a * y * (3 * x * x - y * y), b * x * y * z, e * y * (5 * z * z - 1), f * z * (5 * z * z - 3),
                e * x * (5 * z * z - 1), b / 2 * z * (x * x - y * y), a * x * (x * x - 3 * y * y)]
    return torch.stack(out, -1)


def _geometry(p, cam, opts, degree):
    """Per Gaussian: [n, 18] (projected mean, the forms D, E, X in the offset from it, density, colour), and
    without gradient the rectangle (centre, axis, halves) and whether it is kept."""
    w2c = torch.as_tensor(cam.world_to_cam, device="cuda").double()
    rot, tr = w2c[:, :3], w2c[:, 3]
    q = p["quats"] / p["quats"].norm(dim=1, keepdim=True)
    w, x, y, z = q.unbind(1)
    r = torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y),
                     2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x),
                     2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)], 1).reshape(-1, 3, 3)
    mc = p["means"] @ rot.T + tr
    b = (rot @ r).transpose(1, 2) / p["scales"][:, :, None]
    mg = (b * mc[:, None, :]).sum(2)
    gx, gy, g0 = b[:, :, 0] / cam.fx, b[:, :, 1] / cam.fy, mg / mc[:, 2:]
    px, py = torch.linalg.cross(mg, gx), torch.linalg.cross(mg, gy)
    dot = lambda a, c: (a * c).sum(1)  # noqa: E731
    mean2d = (cam.cx + cam.fx * mc[:, 0] / mc[:, 2], cam.cy + cam.fy * mc[:, 1] / mc[:, 2])
    dd = (dot(g0, g0), dot(gx, g0), dot(gy, g0), dot(gx, gx), dot(gx, gy), dot(gy, gy))
    xx = (dot(px, px), dot(px, py), dot(py, py))
    if degree < 0:
        rgb = p["colors"]
    else:
        view = p["means"] + rot.T @ tr
        basis = _sh_basis(view / view.norm(dim=1, keepdim=True), degree)
        rgb = ((basis[:, :, None] * p["colors"]).sum(1) + 0.5).clamp_min(0)
    coef = torch.stack([*mean2d, *dd, dot(mg, mg) / mc[:, 2], dot(gx, mg), dot(gy, mg), *xx, p["densities"],
                        *rgb.unbind(1)], 1)
    with torch.no_grad():
        quad = dot(mg, mg)
        log_c = math.log(-math.log1p(-opts.conf_c) / math.sqrt(2 * math.pi)) + 0.5 * torch.log(quad / dot(mc, mc))
        delta = 2 * (torch.log(p["densities"]) - log_c)
        qxx, qxy, qyy = (v - delta * u for v, u in zip(xx, dd[3:]))
        det = qxx * qyy - qxy * qxy
        bx, by = delta * dd[1], delta * dd[2]
        cx, cy = (qyy * bx - qxy * by) / det, (qxx * by - qxy * bx) / det
        r2 = delta * dd[0] + bx * cx + by * cy
        keep = (delta > 0) & (delta < quad) & (qxx > 0) & (qyy > 0) & (det > 0) & (r2 > 0)
        big = 0.5 * (qxx + qyy) + torch.sqrt(0.25 * (qxx - qyy) ** 2 + qxy * qxy)
        th = 0.5 * torch.atan2(-qxy, 0.5 * (qyy - qxx))
        rect = torch.stack([mean2d[0] + cx, mean2d[1] + cy, torch.cos(th), torch.sin(th),
                            torch.sqrt(r2 * big / det), torch.sqrt(r2 / big)], 1)
        rad = p["scales"].amax(1)
        keep &= (mc[:, 2] > cam.t_near) & torch.isfinite(rect).all(1)
        for nv in ((cam.fx, 0, cam.cx), (-cam.fx, 0, cam.width - cam.cx), (0, cam.fy, cam.cy),
                   (0, -cam.fy, cam.height - cam.cy)):
            nv = torch.tensor(nv, dtype=torch.float64, device="cuda")
            keep &= (mc @ nv) / nv.norm() + rad >= 0
    return coef, rect, keep


def _boxes(rect, keep, cam):
    """Pixel-centre boxes (x0, x1, y0, y1) of the kept rectangles; x1 < x0 or y1 < y0 where empty."""
    ex = rect[:, 4] * rect[:, 2].abs() + rect[:, 5] * rect[:, 3].abs()
    ey = rect[:, 4] * rect[:, 3].abs() + rect[:, 5] * rect[:, 2].abs()
    lo = lambda v: torch.ceil(v - 0.5).clamp(0, 1e6).nan_to_num(1e6).long()  # noqa: E731
    hi = lambda v, m: torch.floor(v - 0.5).clamp(-1, m - 1).nan_to_num(-1).long()  # noqa: E731
    x0, x1 = lo(rect[:, 0] - ex), hi(rect[:, 0] + ex, cam.width)
    y0, y1 = lo(rect[:, 1] - ey), hi(rect[:, 1] + ey, cam.height)
    return x0, torch.where(keep, x1, -1), y0, y1


def _blocks(boxes, height, most):
    """Row blocks [r0, r1) whose boxes hold about `most` (pixel, Gaussian) candidates."""
    x0, x1, y0, y1 = boxes
    ok = (x1 >= x0) & (y1 >= y0)
    nx = torch.where(ok, x1 - x0 + 1, 0)
    d = torch.zeros(height + 1, dtype=torch.long, device="cuda")
    d.index_add_(0, torch.where(ok, y0, 0), nx)
    d.index_add_(0, torch.where(ok, y1 + 1, 0), -nx)
    rows = torch.cumsum(d, 0)[:height].tolist()
    r0, s = 0, 0
    for r in range(height):
        if s and s + rows[r] > most:
            yield r0, r
            r0, s = r, 0
        s += rows[r]
    yield r0, height


def _pairs_of(rect, boxes, r0, r1):
    """(Gaussian, x, y) of the pixel centres of rows [r0, r1) inside the rectangles."""
    x0, x1, y0, y1 = boxes
    a, b = y0.clamp_min(r0), y1.clamp_max(r1 - 1)
    nx, ny = (x1 - x0 + 1).clamp_min(0), (b - a + 1).clamp_min(0)
    cnt = nx * ny
    ids = torch.nonzero(cnt).squeeze(1)
    cnt = cnt[ids]
    g = torch.repeat_interleave(ids, cnt)
    k = torch.arange(g.numel(), device="cuda") - torch.repeat_interleave(torch.cumsum(cnt, 0) - cnt, cnt)
    x, y = x0[g] + k % nx[g], a[g] + k // nx[g]
    rc = rect[g]
    ax, ay = x + 0.5 - rc[:, 0], y + 0.5 - rc[:, 1]
    inside = ((ax * rc[:, 2] + ay * rc[:, 3]).abs() <= rc[:, 4]) & ((ay * rc[:, 2] - ax * rc[:, 3]).abs() <= rc[:, 5])
    return g[inside], x[inside], y[inside]


def _cholesky(t, m):
    """Lower factor of the Hermitian matrix t(i, j) (lists of tensors) and its pivots."""
    low, piv = [[None] * m for _ in range(m)], []
    for j in range(m):
        s = t(j, j).real
        for k in range(j):
            s = s - (low[j][k] * low[j][k].conj()).real
        piv.append(s)
        low[j][j] = torch.sqrt(s.clamp_min(1e-300))
        for i in range(j + 1, m):
            v = t(i, j)
            for k in range(j):
                v = v - low[i][k] * low[j][k].conj()
            low[i][j] = v / low[j][j]
    return low, piv


def _inverse(low, m):
    inv = [[None] * m for _ in range(m)]
    for i in range(m):
        inv[i][i] = 1.0 / low[i][i]
        for j in range(i):
            inv[i][j] = -sum(low[i][k] * inv[k][j] for k in range(j, i)) / low[i][i]
    return inv


def _mixture(moments, other, t_of, m, rel):
    """The moments, mixed with those of `other` where a Cholesky pivot is below rel times its diagonal."""
    with torch.no_grad():
        level = torch.full_like(moments[0].real, -1.0)
        for e in (0.0,) + MIX:
            c = [(1 - e) * a + e * b for a, b in zip(moments, other)]
            t = t_of(c)
            ok = torch.stack([p > rel * t(j, j).real for j, p in enumerate(_cholesky(t, m)[1])]).all(0)
            level = torch.where((level < 0) & ok, e, level)
        level = level.clamp_min(0)
    return [a + level * (b - a) for a, b in zip(moments, other)]


def _real_roots(c):
    """All roots of a real-rooted polynomial sum_k c[k] x^k of degree 2 to 4, differentiable in c."""
    with torch.no_grad():
        roots, p = [], [v.detach() for v in c]
        while len(p) > 3:  # the root of larger magnitude by Laguerre's iteration from outside all roots
            n = len(p) - 1
            mean = -p[n - 1] / (n * p[n])
            half = torch.sqrt(((n - 1) * ((p[n - 1] / p[n]) ** 2 * (n - 1) / n - 2 * p[n - 2] / p[n]) / n)
                              .clamp_min(0)) * (1 + 1e-9) + 1e-12
            x = torch.where(mean >= 0, mean + half, mean - half)
            for _ in range(24):
                f, d, s = p[n], torch.zeros_like(x), torch.zeros_like(x)
                for v in reversed(p[:n]):
                    s, d, f = s * x + d, d * x + f, f * x + v
                h = torch.sqrt(((n - 1) * ((n - 1) * d * d - 2 * n * f * s)).clamp_min(0))
                step = n * f / torch.where(d >= 0, d + h, d - h)
                x = torch.where(torch.isfinite(step), x - step, x)
            roots.append(x)
            q, prev = [], torch.zeros_like(x)
            for v in p[:n]:  # divided out from the constant term
                prev = (prev - v) / x
                q.append(prev)
            p = q
        h = -0.5 * (p[1] + torch.copysign(torch.sqrt((p[1] * p[1] - 4 * p[0] * p[2]).clamp_min(0)), p[1]))
        roots += [h / p[2], p[0] / h]
    out = []
    for x in roots:
        for last in (False, False, False, True):
            with torch.set_grad_enabled(last and torch.is_grad_enabled()):
                f, d = c[-1], torch.zeros_like(x)
                for v in reversed(c[:-1]):
                    d, f = d * x + f, f * x + v
                step = f / d.detach()
                x = x - torch.where(torch.isfinite(step), step, 0.0)
        out.append(x)
    return out


def _christoffel(inv, powers, m):
    """z = L^-1 v and 1 / |z|^2."""
    z = [sum(inv[i][j] * powers[j] for j in range(i + 1)) for i in range(m)]
    return z, 1.0 / sum((v * v.conj()).real for v in z)


def _bound(inv, s, beta, m):
    """Normalised interpolated moment bound at the standardised query s."""
    z, w0 = _christoffel(inv, [s ** k for k in range(m)], m)
    c = [sum(inv[i][j] * z[i] for i in range(j, m)) for j in range(m)]
    low = torch.zeros_like(s)
    for x in _real_roots(c):
        w = _christoffel(inv, [x ** k for k in range(m)], m)[1]
        low = low + torch.where((x < s) & torch.isfinite(w), w, 0.0)
    return low + beta * w0


def _circle(inv, psi, beta):
    """The canonical representation's estimate on the circle, two complex moments."""
    w = torch.polar(torch.ones_like(psi), psi)
    u, w0 = _christoffel(inv, [w.conj() ** k for k in range(3)], 3)
    a = [sum(inv[i][j].conj() * u[i] for i in range(j, 3)) for j in range(3)]
    sq = torch.sqrt(a[1] * a[1] - 4 * a[0] * a[2])
    sq = torch.where((a[1].conj() * sq).real.detach() < 0, -sq, sq)
    h = -0.5 * (a[1] + sq)
    after = lambda v: torch.remainder(torch.angle(v.detach()) - 1.9 * math.pi, 2 * math.pi)  # noqa: E731
    low = torch.zeros_like(psi)
    for zz in (h / a[2], a[0] / h):
        low = low + torch.where(after(zz) < after(w), _christoffel(inv, [zz.conj() ** k for k in range(3)], 3)[1], 0.0)
    return low + beta * w0


def _network(theta, v):
    """The 7 -> 64 -> 64 -> 1 network (tanh GELU, sigmoid) on rows v [q, 7]."""
    w1, b1, w2, b2, w3, b3 = torch.split(theta, [HIDDEN * INPUTS, HIDDEN, HIDDEN * HIDDEN, HIDDEN, HIDDEN, 1])
    gelu = lambda a: torch.nn.functional.gelu(a, approximate="tanh")  # noqa: E731
    h = gelu(v @ w1.reshape(HIDDEN, INPUTS).T + b1)
    return torch.sigmoid(gelu(h @ w2.reshape(HIDDEN, HIDDEN).T + b2) @ w3 + b3)


def _warp(t, tn):
    return 1 - ((1 + 0.8 * t) / (1 + 0.8 * tn)) ** -1.5


def _warp_d(t, tn):
    return 1.2 * ((1 + 0.8 * t) / (1 + 0.8 * tn)) ** -1.5 / (1 + 0.8 * t)


def _render_rows(case, opts, cam, coef, pairs, r0, r1, theta, want_penalty):
    """Image [rows, W, 3] and penalty [rows, W] of the rows [r0, r1) from their pairs."""
    gid, x, y = pairs
    npx, tn, k = (r1 - r0) * cam.width, cam.t_near, case["moments"]
    f = coef[gid].unbind(1)
    dx, dy = x + 0.5 - f[0], y + 0.5 - f[1]
    lam = torch.sqrt(1 + ((x + 0.5 - cam.cx) / cam.fx) ** 2 + ((y + 0.5 - cam.cy) / cam.fy) ** 2)
    d = f[2] + 2 * (f[3] * dx + f[4] * dy) + f[5] * dx * dx + 2 * f[6] * dx * dy + f[7] * dy * dy
    e = f[8] + f[9] * dx + f[10] * dy
    cross = f[11] * dx * dx + 2 * f[12] * dx * dy + f[13] * dy * dy
    mu, sig, om = lam * e / d, lam / torch.sqrt(d), f[14] * torch.exp(-0.5 * cross / d)
    pix = (y - r0) * cam.width + x
    sums = lambda v: torch.zeros(npx, v.shape[1], dtype=v.dtype, device="cuda").index_add(0, pix, v)  # noqa: E731
    mus = mu.clamp_min(tn)
    a = (tn - mu) / (math.sqrt(2) * sig)
    ea = torch.exp(-a * a)
    mass = om * sig * math.sqrt(math.pi / 2) * torch.special.erfc(a)
    gp = _warp_d(mus, tn)
    if case["trig"]:
        psi0, n = SPAN * (_warp(mus, tn) + gp * (mu - mus)), k // 2
        terms = [torch.complex(mass, torch.zeros_like(mass))]
        for j in range(1, n + 1):
            bj = sig * j * SPAN * gp
            erf = torch.complex(torch.special.erfc(a), bj * math.sqrt(2 / math.pi) * ea)
            amp = om * sig * math.sqrt(math.pi / 2) * torch.exp(-0.5 * bj * bj)
            terms.append(torch.polar(torch.ones_like(amp), j * psi0) * amp * erf)
        acc = sums(torch.stack(terms, 1))
        m0 = acc[:, 0].real
    else:
        with torch.no_grad():  # a moment variable near the pixel's mass (the result does not depend on it)
            st = sums(torch.stack([om * sig, om * sig * mu, om * sig * (mu * mu + sig * sig)], 1))
            ok = st[:, 0] > 0
            mean = torch.where(ok, st[:, 1] / st[:, 0], tn).clamp_min(tn)
            sd = torch.sqrt((st[:, 2] / st[:, 0] - (st[:, 1] / st[:, 0]) ** 2).clamp_min(1e-24))
            org, unit = _warp(mean, tn), torch.where(ok, _warp_d(mean, tn) * sd, 1.0)
        of = lambda t: (_warp(t, tn) - org[pix]) / unit[pix]  # noqa: E731
        yp = gp / unit[pix]
        gg, un, v2 = of(mus) + yp * (mu - mus), of(mus) + yp * (tn - mus), (yp * sig) ** 2
        edge = yp * om * sig * sig * ea
        ms = [mass, gg * mass + edge]
        for j in range(2, k + 1):
            ms.append(gg * ms[-1] + (j - 1) * v2 * ms[-2] + edge * un ** (j - 1))
        acc = sums(torch.stack(ms, 1))
        m0 = acc[:, 0]
    # pixels with depth only from here on; `at` their index per pair
    live = torch.nonzero(m0.detach() > 1e-20).squeeze(1)
    back = torch.full((npx,), -1, dtype=torch.long, device="cuda")
    back[live] = torch.arange(live.numel(), device="cuda")
    sel = back[pix] >= 0
    at = back[pix][sel]
    mu, sig, om, acc = mu[sel], sig[sel], om[sel], acc[live]
    m0l = m0[live]
    m = k // 2 + 1
    if case["trig"]:
        c = [acc[:, j] / m0l for j in range(m)]
        other = [torch.ones_like(c[0])] + [torch.zeros_like(c[0])] * (m - 1)
        toep = lambda v: (lambda i, j: v[i - j].conj() if i >= j else v[j - i])  # noqa: E731
        c = _mixture(c, other, toep, m, 1e-4)
        inv = _inverse(_cholesky(toep(c), m)[0], m)
    else:
        b = [acc[:, j] / m0l for j in range(k + 1)]
        sd = torch.sqrt(b[2] - b[1] * b[1])
        c = [sum(math.comb(i, j) * b[j] * (-b[1]) ** (i - j) for j in range(i + 1)) / sd ** i for i in range(k + 1)]
        hank = lambda v: (lambda i, j: v[i + j])  # noqa: E731
        normal = [torch.full_like(c[0], 0.0 if j % 2 else float(math.prod(range(1, j, 2)))) for j in range(k + 1)]
        mixed = _mixture(c, normal, hank, m, 1e-5)
        inv = _inverse(_cholesky(hank(mixed), m)[0], m)
        feats = torch.asinh(torch.stack(c[1:7], 1)) if theta is not None else None
    ne = case["intervals"] + 1
    quant = [math.sqrt(2) * torch.erfinv(torch.tensor(2 * (j + 0.5) / ne - 1, dtype=torch.float64)).item()
             for j in range(ne)]
    ts = [torch.clamp_min(mu + opts.kappa * q * sig, tn) for q in quant]
    tab = None
    if case["kind"] == "tabulated":
        zs = torch.linspace(-4, 4, NODES, dtype=torch.float64, device="cuda")
        if theta is not None:
            rows = torch.cat([feats[:, None, :].expand(-1, NODES, -1), zs[None, :, None].expand(live.numel(), -1, 1)], 2)
            tab = _network(theta, rows.reshape(-1, INPUTS)).reshape(-1, NODES)
        else:
            tab = torch.stack([_bound(inv, z.expand(live.numel()), opts.beta, m) for z in zs], 1)
    pick = [[v if v is None else v[at] for v in row] for row in inv]
    taus = []
    for t in ts:
        if case["trig"]:
            fv = _circle(pick, SPAN * _warp(t, tn), opts.beta)
        else:
            pt = pix[sel]
            s = ((_warp(t, tn) - org[pt]) / unit[pt] - b[1][at]) / sd[at]
            if tab is not None:
                u = (s.clamp(-4, 4) + 4) * (NODES - 1) / 8
                i0 = u.long().clamp_max(NODES - 2)
                fv = tab[at, i0] + (u - i0) * (tab[at, i0 + 1] - tab[at, i0])
            elif theta is not None:
                fv = _network(theta, torch.cat([feats[at], s.clamp(-10, 10)[:, None]], 1))
            else:
                fv = _bound(pick, s, opts.beta, m)
        taus.append(m0l[at] * fv)
    if case["trig"] or theta is not None or tab is not None:  # estimates need not grow with depth
        taus = list(torch.cummax(torch.stack(taus), 0)[0].unbind(0))
    qs, pen = 0.0, 0.0
    for j in range(ne - 1):
        dt, dtau = ts[j + 1] - ts[j], taus[j + 1] - taus[j]
        phi = torch.where(dtau > 1e-9, -torch.expm1(-dtau) / dtau.clamp_min(1e-9), 1 - 0.5 * dtau)
        qs = qs + torch.exp(-taus[j]) * dt * phi * om * torch.exp(-0.5 * ((ts[j] - mu) / sig) ** 2)
        if want_penalty:
            bs = [(t - mu) / (math.sqrt(2) * sig) for t in (ts[j], ts[j + 1])]
            own = om * sig * math.sqrt(math.pi / 2) * (torch.special.erfc(bs[0]) - torch.special.erfc(bs[1]))
            pen = pen + (own - dtau).clamp_min(0) ** 2
    vals = torch.stack([qs * f[15][sel], qs * f[16][sel], qs * f[17][sel], qs] + ([pen] if want_penalty else []), 1)
    tot = torch.zeros(npx, vals.shape[1], dtype=torch.float64, device="cuda").index_add(0, live[at], vals)
    bg = torch.tensor(cam.background, dtype=torch.float64, device="cuda")
    image = -torch.expm1(-m0)[:, None] * tot[:, :3] / tot[:, 3:4].clamp_min(opts.eps) + torch.exp(-m0)[:, None] * bg
    shape = (r1 - r0, cam.width)
    return image.reshape(*shape, 3), tot[:, 4].reshape(shape) if want_penalty else None


def _view(case, opts, cam, params, theta, back=None):
    """One camera: image [H, W, 3] and penalty [H, W]; `back`(image rows, penalty rows, r0, r1), the scalar whose
    gradient is wanted, makes it add the gradients into the parameters."""
    with torch.set_grad_enabled(back is not None):
        coef, rect, keep = _geometry(params, cam, opts, case["sh"])
        leaf = coef.detach().requires_grad_(back is not None)
    boxes = _boxes(rect, keep, cam)
    want_pen = case["penalty"] or case["kind"] == "train"
    images, pens = [], []
    for r0, r1 in _blocks(boxes, cam.height, 3_000_000 if back is not None or theta is not None else 10_000_000):
        with torch.set_grad_enabled(back is not None):
            img, pen = _render_rows(case, opts, cam, leaf, _pairs_of(rect, boxes, r0, r1), r0, r1, theta, want_pen)
            if back is not None:
                loss = back(img, pen, r0, r1)
                if loss.requires_grad:
                    loss.backward()
        images.append(img.detach())
        pens.append(pen.detach() if want_pen else None)
    if back is not None and leaf.grad is not None:
        coef.backward(leaf.grad)
    return torch.cat(images), torch.cat(pens) if want_pen else None


def _losses(image, target):
    """L1 and 1 - mean SSIM (11 x 11 Gaussian window of 1.5 pixels, zero padding)."""
    win = torch.exp(-torch.arange(-5, 6, dtype=torch.float64, device="cuda") ** 2 / 4.5)
    win = win / win.sum()

    def blur(v):
        v = sum(win[i] * torch.nn.functional.pad(v, (5, 5))[..., i:i + v.shape[-1]] for i in range(11))
        return sum(win[i] * torch.nn.functional.pad(v, (0, 0, 5, 5))[..., i:i + v.shape[-2], :] for i in range(11))

    x, y = image.permute(0, 3, 1, 2), target.permute(0, 3, 1, 2)
    a, b = blur(x), blur(y)
    va, vb, vab = blur(x * x) - a * a, blur(y * y) - b * b, blur(x * y) - a * b
    ssim = (2 * a * b + 1e-4) * (2 * vab + 9e-4) / ((a * a + b * b + 1e-4) * (va + vb + 9e-4))
    return (x - y).abs().mean(), 1 - ssim.mean()


def _adam(p, m, v, g, step, lr):
    m, v = 0.9 * m.double() + 0.1 * g, 0.999 * v.double() + 0.001 * g * g
    return p - lr * (m / (1 - 0.9 ** step)) / (torch.sqrt(v / (1 - 0.999 ** step)) + 1e-8), m, v


def exact(case, seed):
    heavy = 4 * (case["intervals"] + 1) if case["moments"] == 8 else case["intervals"] + 1
    heavy *= 1.0 if case["kind"] in ("frame", "tabulated") else 4.0
    if case["kind"] != "fit" and _pairs(case) * heavy * (20 if case["kind"] == "surrogate" else 1) > 3e9:
        return None  # tens of seconds and more
    s = _inputs(case, seed)
    if case["kind"] == "fit":
        theta = s.theta.double().requires_grad_(True)
        x, t = s.x.double(), s.t.double()
        loss = ((torch.exp(-x[:, 7] * _network(theta, x[:, :INPUTS])) - t) ** 2).mean()
        grad, = torch.autograd.grad(loss, theta)
        new, m, v = _adam(theta.detach(), s.m, s.v, grad, STEP + 1, 1e-3)
        return {"loss": loss.detach().reshape(1), "grad": grad, "theta": new, "m": m, "v": v}
    theta = s.theta.double() if case["kind"] == "surrogate" or case["network"] else None
    grads = case["kind"] in ("step", "autograd", "surrogate", "train")
    params = {k: v.double().requires_grad_(grads) for k, v in s.params.items()}
    if case["kind"] == "train":
        with torch.no_grad():
            image, pen = _view(case, s.opts, s.cams[0], params, theta)
        leaf = image[None].requires_grad_(True)
        l1, ds = _losses(leaf, s.target.double())
        (0.8 * l1 + 0.2 * ds).backward()
        npx = pen.numel()
        _view(case, s.opts, s.cams[0], params, theta,
              lambda img, pn, r0, r1: (img * leaf.grad[0, r0:r1]).sum() + 0.1 * pn.sum() / npx)
        new = {k: _adam(p.detach(), s.m[k], s.v[k], p.grad, STEP + 1, s.lrs[k])[0] for k, p in params.items()}
        l1, ds, cons = l1.detach(), ds.detach(), pen.mean()
        return {"params": new, "l1": l1, "dssim": ds, "consistency": cons, "total": 0.8 * l1 + 0.2 * ds + 0.1 * cons}
    images, pens = [], []
    for i, cam in enumerate(s.cams):
        back = None
        if grads:
            gi, gpen = s.grad_image[i].double(), s.grad_penalty
            back = lambda img, pn, r0, r1: (img * gi[r0:r1]).sum() + (  # noqa: E731
                0.0 if gpen is None else (pn * gpen[i, r0:r1].double()).sum())
        img, pen = _view(case, s.opts, cam, params, theta, back)
        images.append(img)
        pens.append(pen)
    out = {"image": torch.stack(images)}
    if case["kind"] == "frame" and case["penalty"]:
        out["penalty"] = torch.stack(pens)
    if grads:
        out["grads"] = {k: v.grad if v.grad is not None else torch.zeros_like(v) for k, v in params.items()}
    return out
