"""Timing cases: the renderer's work as its users have it done, through the
public entry points of ``paper_2410_08129_amd.htgs``.

A case is a dict of plain values:

``kind``       ``forward`` (inference with a kept workspace), ``noalloc`` (the
               allocation-free inference call), ``train`` (forward and
               backward with kept buffers), ``autograd`` (``htgs.render`` and
               its backward, nothing kept)
``scene``      ``uniform`` (means in [-1, 1]^3, camera 3 units away, fov 60)
               or ``clustered`` (anisotropic clusters, camera 25 units away,
               fov 50), the distributions of ``scenes.py``, drawn on the GPU
``n``, ``sh``  Gaussians and SH degree
``width``, ``height``, ``fov``, ``views``  views above 1 render on a sphere
               around the scene, at four sizes scaled from the given one
``K``, ``tile``, ``cull``, ``order``, ``queue``, ``blend``  render settings;
               ``blend`` is ``ht``, ``no_tail`` or ``sorted``
``baked``, ``filter``, ``densify``, ``degenerate``  input options

Inputs are made from the seed alone. The gradient of the loss with respect to
the image is an input (what the loss of a training program hands over).
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2410_08129_amd import htgs, scenes

_BASE = dict(kind="train", scene="clustered", n=1_000_000, sh=3, width=1920, height=1080,
             fov=50.0, views=1, K=8, tile="8x8", cull=True, order=True, queue=False,
             blend="ht", baked=False, filter=False, densify=False, degenerate=False)


def _case(**kw):
    return {**_BASE, **kw}


def listed():
    return [
        # A thumbnail of a small object: the smallest call, where launches count.
        _case(name="tiny_forward", kind="forward", scene="uniform", n=4096, sh=0, width=128,
              height=128, fov=60.0, K=4, tile="16x16", cull=False, order=False),
        # The same object fitted with the differentiable call, default tile shape.
        _case(name="tiny_autograd", kind="autograd", scene="uniform", n=4096, sh=0, width=128,
              height=128, fov=60.0, K=4, tile="16x16", cull=False, order=False),
        # A viewer that may not allocate, in a window of no particular size.
        _case(name="viewer_noalloc", kind="noalloc", n=60_000, width=803, height=601,
              tile="16x8"),
        # A training step in the middle of densification: 3D filter, densification
        # sums, a core size and an image size that are no powers of two.
        _case(name="densify_step", n=50_001, sh=2, width=637, height=479, K=5, tile="16x16",
              order=False, filter=True, densify=True),
        # The plain differentiable call as documented: default settings but K, no
        # buffers kept.
        _case(name="autograd_800", kind="autograd", n=200_000, sh=3, width=800, height=800,
              tile="16x16", cull=False, order=False),
        # Training at 720p.
        _case(name="train_720p", width=1280, height=720),
        # Training at 1080p (the benchmark's frame).
        _case(name="train_1080p"),
        # Training at 1080p with the core size and, per wave, the tiles that larger
        # cores prefer.
        _case(name="train_1080p_K16", K=16, tile="16x8", queue=True),
        # Frame rate: baked parameters, no tail, no state kept.
        _case(name="baked_1080p", kind="forward", blend="no_tail", baked=True),
        # Training with sorted alpha blending.
        _case(name="sorted_720p", width=1280, height=720, blend="sorted"),
        # Eight views of uneven size in one batched step.
        _case(name="batched_8", n=500_000, width=1280, height=720, views=8, queue=True),
        # The largest frame: 6M Gaussians, some flat, 3840x2160, K = 16.
        _case(name="large_4k", n=6_000_000, width=3840, height=2160, fov=70.0, K=16,
              degenerate=True),
    ]


def draw(rng):
    def log_int(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    kind = rng.choice(("forward", "noalloc", "train", "train", "train", "autograd"))
    scene = "uniform" if rng.random() < 0.2 else "clustered"
    views = rng.randint(2, 6) if kind == "train" and rng.random() < 0.25 else 1
    n = log_int(1000, {"noalloc": 80_000}.get(kind, 30_000 if scene == "uniform" else 2_000_000))
    width = log_int(72, 1000 if kind == "noalloc" or scene == "uniform" else 2560)
    height = max(40, min(1440, int(width * rng.uniform(0.5, 1.3))))
    if views > 1:
        n, width, height = min(n, 400_000), min(width, 1280), min(height, 800)
    tile = rng.choice(("8x8", "8x8", "16x8", "16x16", "32x8"))
    K = rng.choice((1, 2, 3, 4, 6, 8, 8, 8, 12, 16, 16, 24, 32))
    if tile in ("16x16", "32x8"):
        K = min(K, 16)
    blend = "ht"
    if kind == "forward":
        blend = rng.choice(("ht", "no_tail", "sorted"))
    elif kind == "train" and views == 1 and rng.random() < 0.25:
        blend = "sorted"
    baked = kind in ("forward", "noalloc") and rng.random() < 0.4
    return _case(kind=kind, scene=scene, n=n, sh=rng.randint(0, 3), width=width, height=height,
                 fov=round(rng.uniform(45.0, 70.0), 1), views=views, K=K, tile=tile,
                 cull=rng.random() < 0.6, order=rng.random() < 0.5, queue=rng.random() < 0.3,
                 blend=blend, baked=baked, filter=not baked and rng.random() < 0.25,
                 densify=kind == "train" and rng.random() < 0.3,
                 degenerate=rng.random() < 0.2)


# ---------------------------------------------------------------------------
# Inputs
# ---------------------------------------------------------------------------

def _scene(case, seed):
    """Parameters (means, log-scales, quaternions, logits, SH) on the GPU, and the
    filter variance or None."""
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev)
    gen.manual_seed(int(seed))
    n, nb = case["n"], (case["sh"] + 1) ** 2

    def normal(*shape):
        return torch.randn(*shape, generator=gen, device=dev)

    def uniform(*shape):
        return torch.rand(*shape, generator=gen, device=dev)

    if case["scene"] == "uniform":
        means = 2.0 * uniform(n, 3) - 1.0
        ls = -4.0 + 0.5 * normal(n, 3)
        logits = normal(n)
    else:
        centres = 20.0 * uniform(64, 3) - 10.0
        cid = torch.randint(0, 64, (n,), generator=gen, device=dev)
        means = centres[cid] + normal(n, 3) * torch.tensor([2.0, 0.5, 2.0], device=dev)
        ls = -3.5 + 0.7 * normal(n, 3)
        logits = 1.5 * normal(n)
    quats = torch.nn.functional.normalize(normal(n, 4), dim=1)
    sh = 0.05 * normal(n, nb, 3)
    sh[:, 0] = (uniform(n, 3) - 0.5) / (0.5 / math.sqrt(math.pi))
    if case["degenerate"]:
        # 10% with one zero axis, 2% with one axis of scale 1e-7
        u, axis = uniform(n), torch.randint(0, 3, (n,), generator=gen, device=dev)
        pick = torch.nn.functional.one_hot(axis, 3).bool()
        ls = torch.where(pick & (u < 0.10)[:, None], torch.full_like(ls, -math.inf), ls)
        ls = torch.where(pick & ((u >= 0.10) & (u < 0.12))[:, None],
                         torch.full_like(ls, math.log(1e-7)), ls)
    fv = None
    if case["filter"]:
        fv = (0.3 * torch.exp(-3.5 + 0.3 * normal(n))) ** 2
    if case["baked"]:
        ls, logits = torch.exp(ls), torch.sigmoid(logits)
    params = [means, ls, quats, logits, sh]
    return [p.contiguous() for p in params], fv


def _cameras(case, seed):
    r = 3.0 if case["scene"] == "uniform" else 25.0
    if case["views"] == 1:
        return [scenes.look_at((0, 0, -r), (0, 0, 0), (0, -1, 0), case["fov"], case["width"],
                               case["height"])]
    rng = np.random.default_rng(int(seed))
    cams = []
    for v in range(case["views"]):
        e = rng.normal(0.0, 1.0, 3)
        e[1] *= 0.5
        e = r * e / np.linalg.norm(e)
        f = (1.0, 0.5, 0.75, 0.8)[v % 4]
        cams.append(scenes.look_at(e, (0, 0, 0), (0, -1, 0), case["fov"],
                                   max(8, int(case["width"] * f)), max(8, int(case["height"] * f))))
    return cams


def _settings(case):
    tw, th = (int(x) for x in case["tile"].split("x"))
    return scenes.RenderSettings(
        K=case["K"], tile_w=tw, tile_h=th, tile_cull=case["cull"], cost_order=case["order"],
        persistent=case["queue"], no_tail=case["blend"] == "no_tail",
        sorted_blend=case["blend"] == "sorted", baked=case["baked"],
        bg=(0.1, 0.2, 0.3), grad_overwrite=case["kind"] == "train" and case["views"] == 1
        and not case["densify"])


def _image_grads(case, cams, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed) + 7_654_321)
    return [torch.randn(3, c.height, c.width, generator=gen, device="cuda") / (3 * c.height * c.width)
            for c in cams]


def prepare(case, seed):
    params, fv = _scene(case, seed)
    cams, st = _cameras(case, seed), _settings(case)
    full = params + ([fv] if fv is not None else [])
    s = dict(case=case, params=params, full=full, fv=fv, cams=cams, st=st, sh=case["sh"])
    images = [torch.empty((3, c.height, c.width), device="cuda") for c in cams]
    if case["kind"] == "noalloc":
        s.update(image=images[0], status=torch.zeros(1, dtype=torch.int32, device="cuda"))
        return s
    if case["kind"] == "autograd":
        s.update(params=[p.requires_grad_(True) for p in params],
                 gimg=_image_grads(case, cams, seed)[0])
        return s
    count = htgs.count_instances(full, case["sh"], cams, st)
    s.update(images=images, ws=htgs.alloc_workspace(case["n"], cams, st, count, params[0].device))
    if case["kind"] == "train":
        s.update(state=torch.empty(htgs.state_bytes(cams, st) // 4, device="cuda"),
                 gimgs=_image_grads(case, cams, seed),
                 # kept gradients where the backward writes them; where it adds,
                 # each step starts from new zeros
                 grads=[torch.zeros_like(p) for p in params] if st.grad_overwrite else None,
                 densify=tuple(torch.zeros(case["n"], device="cuda") for _ in range(2))
                 if case["densify"] else None)
    return s


_NAMES = ("means", "log_scales", "quats", "logits", "sh")


def run(s):
    kind = s["case"]["kind"]
    if kind == "noalloc":
        htgs.forward_noalloc(s["full"], s["sh"], s["cams"][0], s["st"], s["image"],
                             status=s["status"])
        return {"images": [s["image"]], "status": s["status"]}
    if kind == "autograd":
        img = htgs.render(*s["params"], s["sh"], s["cams"][0], s["st"], filter_var=s["fv"])
        grads = torch.autograd.grad(img, s["params"], s["gimg"])
        return {"images": [img.detach()], "grads": dict(zip(_NAMES, grads))}
    if kind == "forward":
        frame = htgs.forward(s["full"], s["sh"], s["cams"], s["st"], ws=s["ws"],
                             images=s["images"], with_state=False)
        return {"images": frame.images}
    frame = htgs.forward(s["full"], s["sh"], s["cams"], s["st"], ws=s["ws"], state=s["state"],
                         images=s["images"])
    grads = htgs.backward(s["full"], frame, s["gimgs"], grads=s["grads"], densify=s["densify"])
    out = {"images": frame.images, "grads": dict(zip(_NAMES, grads))}
    if s["densify"] is not None:
        out["densify"] = list(s["densify"])
    return out


# ---------------------------------------------------------------------------
# Work
# ---------------------------------------------------------------------------

def work(case):
    """Bytes: the parameters read once (once more by a backward) and the images and
    gradients written once. Flops: an estimate of the pixel-Gaussian fragments
    (from the mean squared scale and the focal length) times the arithmetic of one:
    the two norms and the cutoff test (25), alpha and the blend (15), and for a
    backward the same test, the adjoints and the moments (90)."""
    grad = case["kind"] in ("train", "autograd")
    floats = 11 + 3 * (case["sh"] + 1) ** 2
    px = frags = 0.0
    sizes = [(1.0, 0.5, 0.75, 0.8)[v % 4] if case["views"] > 1 else 1.0
             for v in range(case["views"])]
    # fragments of a Gaussian at fov 50 and 1920 pixels: 194 (clustered scene);
    # the uniform scene is nearer and its Gaussians smaller: about five times that
    per = (194.0 if case["scene"] == "clustered" else 1000.0) * \
        (math.tan(math.radians(25.0)) / math.tan(math.radians(case["fov"] / 2.0))) ** 2
    for f in sizes:
        px += case["width"] * case["height"] * f * f
        frags += case["n"] * per * (case["width"] * f / 1920.0) ** 2
    nbytes = 4.0 * case["n"] * floats * (3 if grad else 1) + 12.0 * px * (2 if grad else 1)
    return {"bytes": nbytes, "flops": frags * (130.0 if grad else 40.0)}


# ---------------------------------------------------------------------------
# The same in 64 bits: every Gaussian at every pixel of the blocks its box meets
# ---------------------------------------------------------------------------

def _rotations(q):
    w, x, y, z = (q / q.norm(dim=1, keepdim=True)).unbind(1)
    return torch.stack([
        torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y - w * z), 2 * (x * z + w * y)], 1),
        torch.stack([2 * (x * y + w * z), 1 - 2 * (x * x + z * z), 2 * (y * z - w * x)], 1),
        torch.stack([2 * (x * z - w * y), 2 * (y * z + w * x), 1 - 2 * (x * x + y * y)], 1)], 1)


def _harmonics(d, degree):
    """Orthonormal real spherical harmonics without the Condon-Shortley phase."""
    x, y, z = d.unbind(1)
    pi = math.pi
    b = [torch.full_like(x, 0.5 / math.sqrt(pi))]
    if degree >= 1:
        c = math.sqrt(3 / (4 * pi))
        b += [c * y, c * z, c * x]
    if degree >= 2:
        c = math.sqrt(15 / pi) / 2
        b += [c * x * y, c * y * z, math.sqrt(5 / pi) / 4 * (3 * z * z - 1), c * x * z,
              c / 2 * (x * x - y * y)]
    if degree >= 3:
        a, c, e = math.sqrt(35 / (2 * pi)) / 4, math.sqrt(105 / pi) / 2, math.sqrt(21 / (2 * pi)) / 4
        b += [a * y * (3 * x * x - y * y), c * x * y * z, e * y * (5 * z * z - 1),
              math.sqrt(7 / pi) / 4 * z * (5 * z * z - 3), e * x * (5 * z * z - 1),
              c / 2 * z * (x * x - y * y), a * x * (x * x - 3 * y * y)]
    return torch.stack(b, 1)


def _splats(case, p, fv, cam, st):
    """Per Gaussian: opacity, cutoff, rows of the view transform, centre, colour, and
    which of them the camera can see."""
    means, ls, quats, logits, sh = p
    scale, o = (ls, logits) if case["baked"] else (torch.exp(ls), torch.sigmoid(logits))
    if fv is not None:
        wide = torch.sqrt(scale * scale + fv.double()[:, None])
        o, scale = o * (scale / wide).prod(1), wide
    w2c = torch.tensor(np.asarray(cam.world_to_cam, np.float64), device=means.device)
    W, t = w2c[:, :3], w2c[:, 3]
    R = _rotations(quats)
    rows = (W @ R) * scale[:, None, :]
    mv = means @ W.T + t
    rc = 2.0 * torch.log(o / float(np.float32(st.tau_alpha)))
    seen = (o > float(np.float32(st.tau_alpha))) & (mv[:, 2] > float(np.float32(cam.z_near)))
    seen = seen & (rc * (rows[:, 2] ** 2).sum(1) < mv[:, 2] ** 2)
    centre = torch.tensor(cam.center, device=means.device)
    d = torch.nn.functional.normalize(means - centre, dim=1)
    colour = torch.clamp((_harmonics(d, case["sh"])[:, :, None] * sh).sum(1) + 0.5, min=0.0)
    return o, rc, rows, mv, colour, seen


def _pixels(o, rc, rows, mv, colour, st, cam, x, y):
    """Colours [pixels, 3] of the pixels (x, y) for the given splats."""
    u = ((x + 0.5 - float(np.float32(cam.cx))) / float(np.float32(cam.fx)))[:, None, None]
    v = ((y + 0.5 - float(np.float32(cam.cy))) / float(np.float32(cam.fy)))[:, None, None]
    a, b = rows[None, :, 0] - u * rows[None, :, 2], rows[None, :, 1] - v * rows[None, :, 2]
    a0, b0 = mv[None, :, 0:1] - u * mv[None, :, 2:3], mv[None, :, 1:2] - v * mv[None, :, 2:3]
    d, m = torch.linalg.cross(a, b), a0 * b - b0 * a
    dd, mm = (d * d).sum(2), (m * m).sum(2)
    hit = dd > 0
    dd = torch.where(hit, dd, torch.ones_like(dd))
    rho2 = mm / dd
    hit = hit & (rho2 <= rc[None])
    alpha = torch.clamp(o[None] * torch.exp(-0.5 * rho2), max=float(np.float32(st.alpha_max)))
    alpha = torch.where(hit, alpha, torch.zeros_like(alpha))
    bg = torch.tensor([float(np.float32(c)) for c in st.bg], dtype=torch.float64, device=o.device)
    if st.sorted_blend:
        # (the splats come front to back)
        T = torch.cumprod(1.0 - alpha, 1)
        live = torch.cumsum((hit & (T < float(np.float32(st.tau_T)))).long(), 1) == 0
        alpha = torch.where(live, alpha, torch.zeros_like(alpha))
        T = torch.cumprod(1.0 - alpha, 1)
        before = torch.cat([torch.ones_like(T[:, :1]), T[:, :-1]], 1)
        return (alpha * before) @ colour + T[:, -1:] * bg
    z = (torch.linalg.cross(d, m) * rows[None, :, 2]).sum(2) / dd + mv[None, :, 2]
    eligible = hit & (alpha >= float(np.float32(st.tau_core)))
    k = min(st.K, alpha.shape[1])
    front = torch.where(eligible, z, torch.full_like(z, math.inf)).detach()
    zs, at = front.topk(k, 1, largest=False, sorted=True)
    got = torch.isfinite(zs)
    core = torch.where(got, alpha.gather(1, at), torch.zeros_like(zs))
    T = torch.cumprod(1.0 - core, 1)
    before = torch.cat([torch.ones_like(T[:, :1]), T[:, :-1]], 1)
    C = ((core * before)[:, :, None] * colour[at]).sum(1)
    last = T[:, -1:] if k else torch.ones_like(C[:, :1])
    if st.no_tail:
        return C + last * bg
    rest = alpha.scatter(1, at, torch.where(got, torch.zeros_like(core), alpha.gather(1, at)))
    A, S, P = rest.sum(1, keepdim=True), rest @ colour, (1.0 - rest).prod(1, keepdim=True)
    tail = torch.where(A > 0, (1.0 - P) * S / torch.where(A > 0, A, torch.ones_like(A)), 0.0 * S)
    return C + last * (tail + P * bg)


_BLOCK = 32


def _boxes(rc, rows, mv, cam):
    """Screen boxes of the cutoff ellipsoids, widened by a pixel: [n, 4] (x0, x1, y0, y1)."""
    fx, fy, cx, cy = (float(np.float32(c)) for c in (cam.fx, cam.fy, cam.cx, cam.cy))
    last, l0 = rows[:, 2], mv[:, 2]
    s = rc * (last * last).sum(1) - l0 * l0
    out = []
    for row, r0 in ((fx * rows[:, 0] + cx * last, fx * mv[:, 0] + cx * l0),
                    (fy * rows[:, 1] + cy * last, fy * mv[:, 1] + cy * l0)):
        p = (rc * (row * last).sum(1) - r0 * l0) / s
        q = (rc * (row * row).sum(1) - r0 * r0) / s
        h = torch.sqrt(torch.clamp(p * p - q, min=0.0))
        out += [p - h - 1.5, p + h + 0.5]
    return torch.stack(out, 1)


@torch.no_grad()
def _blocks(box, cam):
    """(block, splat) pairs in block order, splats in their own order inside a block, as
    the splat indices and the end of each block's run."""
    bw, bh = -(-cam.width // _BLOCK), -(-cam.height // _BLOCK)
    lo = torch.clamp(torch.floor(box[:, ::2] / _BLOCK), min=0).long()
    hi = torch.floor(box[:, 1::2] / _BLOCK)
    hi = torch.minimum(hi, torch.tensor([bw - 1.0, bh - 1.0], device=hi.device)).long()
    size = torch.clamp(hi - lo + 1, min=0)
    count = size[:, 0] * size[:, 1]
    who = torch.repeat_interleave(torch.arange(len(box), device=box.device), count)
    k = torch.arange(len(who), device=box.device) - (torch.cumsum(count, 0) - count)[who]
    block = (lo[who, 1] + k // size[who, 0]) * bw + lo[who, 0] + k % size[who, 0]
    block, order = block.sort(stable=True)
    return who[order], torch.cumsum(torch.bincount(block, minlength=bw * bh), 0).tolist()


def exact(case, seed):
    grad = case["kind"] in ("train", "autograd")
    # (flat Gaussians: the rasterizer's own rounding decides which rays they meet)
    if case["n"] * case["views"] > 2_500_000 or (grad and case["degenerate"]):
        return None
    params, fv = _scene(case, seed)
    cams, st = _cameras(case, seed), _settings(case)
    p = [x.double().requires_grad_(grad) for x in params]
    images = []
    left = 5_000_000_000   # pixel-Gaussian pairs: about 20 seconds
    for cam, gimg in zip(cams, _image_grads(case, cams, seed)):
        splats = _splats(case, p, fv, cam, st)
        seen = torch.nonzero(splats[-1])[:, 0]
        if st.sorted_blend:
            seen = seen[splats[3][seen, 2].detach().float().sort(stable=True)[1]]
        kept = [s[seen] for s in splats[:-1]]
        cut = [k.detach() for k in kept]
        sums = [torch.zeros_like(k) for k in cut] if grad else None
        who, ends = _blocks(_boxes(cut[1], cut[2], cut[3], cam), cam)
        left -= len(who) * _BLOCK * _BLOCK
        if left < 0:
            return None
        bg = torch.tensor([float(np.float32(c)) for c in st.bg], dtype=torch.float64, device="cuda")
        img = bg[:, None, None].repeat(1, cam.height, cam.width)
        bw, begin = -(-cam.width // _BLOCK), 0
        for b, end in enumerate(ends):
            at, begin = who[begin:end], end
            x0, y0 = b % bw * _BLOCK, b // bw * _BLOCK
            w, h = min(_BLOCK, cam.width - x0), min(_BLOCK, cam.height - y0)
            rows = max(1, min(h, 8_000_000 // max(1, len(at) * w)))
            if not len(at):
                continue
            sub = [k[at].requires_grad_(grad) for k in cut]
            for y1 in range(y0, y0 + h, rows):
                hh = min(rows, y0 + h - y1)
                k = torch.arange(w * hh, device="cuda")
                c = _pixels(*sub, st, cam, (x0 + k % w).double(), (y1 + k // w).double())
                img[:, y1:y1 + hh, x0:x0 + w] = c.detach().T.reshape(3, hh, w)
                if grad:
                    (c.T.reshape(3, hh, w) * gimg[:, y1:y1 + hh, x0:x0 + w]).sum().backward()
            if grad:
                for t, k in zip(sums, sub):
                    if k.grad is not None:
                        t.index_add_(0, at, k.grad)
        images.append(img)
        if grad:
            torch.autograd.backward(kept, sums)
    out = {"images": images}
    if case["kind"] == "noalloc":
        out["status"] = None
    if grad:
        out["grads"] = dict(zip(_NAMES, [x.grad for x in p]))
    if case["densify"]:
        out["densify"] = [None, None]
    return out
