"""The work this rasterizer is used for, as measurable cases: training steps, single views, the autograd
path, the lists, the training loss, the significance score and the progressive targets.

`listed()` names the cases, `draw(rng)` gives one more of the same ranges, `prepare(case, seed)` makes what
a program holds before the call (parameters, targets, the Rasterizer or Step it keeps), `run(state)` is one
pass through the public entry points, `work(case)` the bytes and operations a pass cannot do without, and
`exact(case, seed)` the same outputs in 64 bits from plain torch, for the sizes where that takes seconds.

Scenes follow the workloads of `paper_2501_14534_amd.scenes` (same distributions, drawn on the GPU):
  cube   U[-1,1]^3 before one camera            (the 2K-Gaussian workload)
  shell  unit directions x U[0.6,1]             (200K and 1M Gaussians, ring of cameras)
  box    normal, kept inside a box              (1M masked Gaussians)
  room   uniform box with the cameras inside it (6M Gaussians)
"""
import math

import numpy as np
import torch

from paper_2501_14534_amd import progressive, raster, scenes
from paper_2501_14534_amd.photometric import PhotometricLoss

LAMBDA_MASK = (0.05, 0.05)  # Eq. 7's mask weights (Sec. 4.2)
LAMBDA_SSIM = 0.2

# log-scale (mean, sd) and opacity-logit (mean, sd) of the scene kinds
SHAPES = {"cube": ((-3.5, 0.4), (0.0, 1.0)), "shell": ((-4.5, 0.5), (0.0, 1.5)),
          "box": ((-3.8, 0.7), (0.0, 1.0)), "room": ((-3.5, 0.8), (-0.5, 1.5))}

MIXED = "316x208,632x416,1264x832,316x208,632x416,1264x832,316x208,632x416"
LARGE = "1920x1080,1920x1080,1920x1080,1920x1080,960x540,960x540,960x540,960x540"


def _case(name, do, scene, n, deg, views, tile="16x16", ppt=1, bwd_chunk=512, masks=False, band_masks=False,
          loss="l2", graph=True, sh_rest=True, progressive_lowpass=False):
    c = dict(do=do, scene=scene, n=n, deg=deg, views=views, tile=tile, ppt=ppt, bwd_chunk=bwd_chunk, masks=masks,
             band_masks=band_masks, loss=loss, graph=graph, sh_rest=sh_rest, progressive_lowpass=progressive_lowpass)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # a captured training step on a toy scene: launches and latency are all there is
        _case("step_2k_128", "step", "cube", 2000, 0, "128x128", tile="16x8", bwd_chunk=1024),
        # a captured training step on one object-sized scene and one view (a step of the 3DGS schedule)
        _case("step_200k_800", "step", "shell", 200_000, 3, "800x800", bwd_chunk=256),
        # the benchmark: eight progressive-resolution views of 1M masked Gaussians in one captured step
        _case("step_1m_8views", "step", "shell", 1_000_000, 3, MIXED, masks=True, band_masks=True),
        # the paper's whole objective (Eq. 7: L1 + D-SSIM + mask terms) on one full-resolution view
        _case("step_1m_dssim", "step", "box", 1_000_000, 3, "1600x1064", tile="32x16", ppt=2, bwd_chunk=256,
              masks=True, band_masks=True, loss="l1_dssim"),
        # the largest scene of the paper's range (6M Gaussians), eight views up to 1080p
        _case("step_6m_8views", "step", "room", 6_000_000, 3, LARGE, tile="32x32", ppt=4, bwd_chunk=1024,
              band_masks=True),
        # viewing a trained scene: one full-resolution frame, forward only, with the overflow check
        _case("view_1m_1600", "view", "box", 1_000_000, 3, "1600x1064"),
        # a thumbnail frame of a pruned scene, an odd size: latency of the forward calls
        _case("view_20k_333", "view", "shell", 20_000, 1, "333x217"),
        # a research loop through torch.autograd: ragged views, both kinds of mask, eager
        _case("autograd_30k_ragged", "autograd", "shell", 30_000, 3, "401x299,203x151,97x73", masks=True,
              band_masks=True, graph=False),
        # projection and the depth-ordered tile lists alone (what inspection and pruning tools call)
        _case("lists_1m_8views", "lists", "shell", 1_000_000, 3, MIXED, masks=True, band_masks=True),
        # the photometric loss and its gradient on the benchmark's views
        _case("loss_8views", "loss", "shell", 1000, 0, MIXED),
        # the significance score of Eq. 4 over a batch of training views, as a pruning pass calls it
        _case("score_1m_8views", "score", "shell", 1_000_000, 3, MIXED, masks=True, band_masks=True),
        # the targets of progressive training: resize to the current resolution, blur at full size
        _case("targets_3views", "targets", "shell", 1000, 0, "1264x832,800x800,633x417"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: kind, scene, sizes (log-uniform, odd ones among them), degree, masks and launch shape."""
    do = rng.choice(["step", "step", "step", "step", "view", "view", "autograd", "lists", "loss", "score", "targets"])
    scene = rng.choice(["cube", "shell", "shell", "box", "room"])
    n_max = {"step": 6_000_000, "view": 3_000_000, "autograd": 1_000_000, "lists": 2_000_000, "loss": 1000,
             "score": 1_500_000, "targets": 1000}[do]
    n = _log_int(rng, 1500, n_max) if n_max > 1000 else 1000
    if scene in ("cube", "box") and n > 500_000:
        scene = "room"  # dense scenes stay at the counts they are drawn for
    nv = rng.choice([1, 1, 2, 3, 5, 8])
    if n * nv > 24_000_000:
        nv = 1
    sizes = []
    for _ in range(nv):
        w = _log_int(rng, 96, 1920)
        sizes.append("%dx%d" % (w, max(64, int(w * rng.choice([0.5625, 0.658, 0.665, 1.0])))))
    tile, ppt = rng.choice([("16x16", 1), ("16x16", 1), ("16x8", 1), ("32x16", 2), ("32x32", 4)])
    masks = rng.random() < 0.5
    deg = rng.choice([0, 1, 2, 3, 3, 3])
    band_masks = deg > 0 and rng.random() < 0.6 and (do != "autograd" or deg == 3)
    return _case(None, do, scene, n, deg, ",".join(sizes), tile=tile, ppt=ppt,
                 bwd_chunk=rng.choice([256, 512, 512, 1024]), masks=masks,
                 band_masks=band_masks, loss=rng.choice(["l2", "l2", "l1_dssim"]),
                 graph=do == "step" and rng.random() < 0.8, sh_rest=rng.random() < 0.75,
                 progressive_lowpass=rng.random() < 0.2)


# ---------------------------------------------------------------------------
# inputs


def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _sizes(case):
    return [tuple(int(x) for x in s.split("x")) for s in case["views"].split(",")]


def _cams(case):
    """The views of the case's scene kind; poses depend on the view's index alone."""
    sizes, cams = _sizes(case), []
    poses = np.random.default_rng(5)
    for v, (w, h) in enumerate(sizes):
        kind = case["scene"]
        if kind == "room":
            pos = poses.uniform([-24.0, -24.0, -8.0], [24.0, 24.0, 8.0])
            yaw, pitch = poses.uniform(0.0, 2.0 * math.pi), math.radians(poses.uniform(-10.0, 10.0))
            fwd = np.array([math.cos(pitch) * math.cos(yaw), math.cos(pitch) * math.sin(yaw), math.sin(pitch)])
            cams.append(scenes.make_camera(pos, pos + fwd, w, h, 1500.0 * max(w, 960) / 1920.0))
            continue
        th = 2.0 * math.pi * v / max(len(sizes), 1)
        if kind == "cube":
            r, z, f = 4.0, 0.0, float(w)
        elif kind == "box":
            r, z, f = 8.0, 1.0, w * 1200.0 / 1600.0
        else:
            r, z, f = (8.0, 0.0, w * 1111.0 / 800.0) if len(sizes) > 1 else (4.0, 0.0, w * 1111.0 / 800.0)
        cams.append(scenes.make_camera((r * math.sin(th), -r * math.cos(th), z), (0, 0, 0), w, h, f))
    return cams


def _opts(case):
    tw, th = (int(x) for x in case["tile"].split("x"))
    return scenes.Opts(tile_w=tw, tile_h=th, pixels_per_thread=case["ppt"], bwd_chunk=case["bwd_chunk"],
                       lowpass_progressive=int(case["progressive_lowpass"]))


def _params(case, seed):
    """Raw Gaussian parameters of the case's scene, drawn on the device from the seed."""
    dev, n = _device(), case["n"]
    g = torch.Generator(device=dev).manual_seed(1_000_003 * int(seed) + 17)

    def normal(mean, sd, *shape):
        return torch.randn(*shape, generator=g, device=dev).mul_(sd).add_(mean)

    def uniform(lo, hi, *shape):
        return torch.rand(*shape, generator=g, device=dev).mul_(hi - lo).add_(lo)

    kind = case["scene"]
    if kind == "cube":
        means = uniform(-1.0, 1.0, 3, n)
    elif kind == "shell":
        d = normal(0.0, 1.0, 3, n)
        means = d / d.norm(dim=0, keepdim=True) * uniform(0.6, 1.0, n)
    elif kind == "box":
        sd = torch.tensor([5.0, 5.0, 2.5], device=dev)[:, None]
        means = torch.fmod(normal(0.0, 1.0, 3, n), 2.0) * sd
    else:
        means = uniform(-1.0, 1.0, 3, n) * torch.tensor([30.0, 30.0, 10.0], device=dev)[:, None]
    (lm, ls), (om, os_) = SHAPES[kind]
    q = normal(0.0, 1.0, 4, n)
    p = dict(means=means.contiguous(), log_scales=normal(lm, ls, 3, n), quats=(q / q.norm(dim=0, keepdim=True)).contiguous(),
             opacity_logits=normal(om, os_, n), sh_dc=normal(0.5, 0.2, 3, n))
    if case["deg"] > 0:
        p["sh_rest"] = normal(0.0, 0.05, (case["deg"] + 1) ** 2 - 1, 3, n)
    if case["masks"]:
        p["mask_logits"] = normal(0.0, 1.0, n)
    if case["band_masks"] and case["deg"] > 0:
        p["sh_mask_logits"] = normal(0.0, 1.0, 3, n)
    return p


def _planes(case, seed):
    """Images in [0, 1], views concatenated: smooth content with noise, as photographs have."""
    dev = _device()
    g = torch.Generator(device=dev).manual_seed(7_000_003 * int(seed) + 29)
    out = []
    for w, h in _sizes(case):
        low = torch.rand(1, 3, max(2, h // 16), max(2, w // 16), generator=g, device=dev)
        img = torch.nn.functional.interpolate(low, size=(h, w), mode="bilinear", align_corners=False)[0]
        img = img + 0.05 * torch.randn(3, h, w, generator=g, device=dev)
        out.append(img.clamp_(0.0, 1.0).reshape(-1))
    return torch.cat(out)


def _rasterizer(case, capacity=None):
    return raster.Rasterizer(case["n"], case["deg"], _cams(case), _opts(case), capacity=capacity)


def prepare(case, seed):
    do, s = case["do"], dict(case=case)
    if do == "step":
        s["step"] = raster.Step(_rasterizer(case), _params(case, seed), _planes(case, seed), graph=case["graph"],
                                loss=case["loss"], mask_loss=LAMBDA_MASK if case["loss"] == "l1_dssim" else None)
        s["step"].run()  # sizes the lists; captures the graph
        if not case["sh_rest"]:
            s["step"].launch(False)
    elif do == "view":
        s["rast"], s["params"] = _rasterizer(case), _params(case, seed)
        s["rast"].forward(s["params"])  # sizes the lists
    elif do == "autograd":
        s["rast"] = _rasterizer(case)
        s["params"] = {k: v.requires_grad_(True) for k, v in _params(case, seed).items()}
        s["weight"] = _planes(case, seed)
        raster.rasterize(s["rast"], s["params"])
    elif do == "lists":
        # lists of a fixed size, doubled until the pairs fit (the whole buffers are the outputs)
        capacity = max(1 << 16, 5 * case["n"] * len(_sizes(case)) // 2)
        while True:
            s["rast"], s["params"] = _rasterizer(case, capacity), _params(case, seed)
            s["rast"].project(s["params"])
            s["rast"].bin_sort()
            if not s["rast"].overflowed():
                break
            capacity *= 2
    elif do == "loss":
        s["loss"] = PhotometricLoss(_cams(case), LAMBDA_SSIM)
        s["image"], s["target"] = _planes(case, seed), _planes(case, seed + 500_000)
    elif do == "score":
        s["params"], s["cams"], s["opts"] = _params(case, seed), _cams(case), _opts(case)
    elif do == "targets":
        img, cams = _planes(case, seed), _cams(case)
        s["resize"] = progressive.ProgressiveTargets(img, cams)              # 8x smaller at the start
        s["blur"] = progressive.ProgressiveTargets(img, cams, start=1.0)     # full size, 9 x 9 at the start
    else:
        raise ValueError(do)
    return s


# ---------------------------------------------------------------------------
# one pass


def run(s):
    case = s["case"]
    do = case["do"]
    if do == "step":
        st = s["step"]
        st.launch(case["sh_rest"])
        out = dict(image=st.rast.image, grads=dict(st.grads))
        if st.ploss is not None:
            out["loss"], out["mask_loss"] = st.ploss.loss, st.mask_value
        return out
    if do == "view":
        return dict(image=s["rast"].forward(s["params"]))
    if do == "autograd":
        img = raster.rasterize(s["rast"], s["params"])
        names = list(s["params"])
        grads = torch.autograd.grad((img * s["weight"]).sum(), [s["params"][k] for k in names])
        return dict(image=img.detach(), grads=dict(zip(names, grads)))
    if do == "lists":
        r = s["rast"]
        r.project(s["params"])
        r.bin_sort()
        return dict(splats=r.splat_records(), tiles_touched=r.tiles_touched, offsets=r.offsets, ids=r.ids,
                    pair_index=r.pair_index, ranges=r.ranges, count=r.count)
    if do == "loss":
        loss, grad = s["loss"](s["image"], s["target"])
        return dict(loss=loss, grad=grad)
    if do == "score":
        return raster.significance_scores(s["params"], case["deg"], s["cams"], s["opts"])
    small, blurred = s["resize"].at(1000), s["blur"].at(1000)
    return dict(small=small[1], blurred=blurred[1])


def _param_floats(case):
    k = (case["deg"] + 1) ** 2 - 1
    return 14 + 3 * k + int(case["masks"]) + (3 if case["band_masks"] and case["deg"] > 0 else 0)


def work(case):
    """Parameters, targets, images, gradients and lists moved once; projection arithmetic per record and
    compositing arithmetic for some ten Gaussians a pixel (an order of magnitude: the scene decides)."""
    n, sizes = case["n"], _sizes(case)
    px, nrec, par = sum(w * h for w, h in sizes), case["n"] * len(sizes), _param_floats(case)
    do = case["do"]
    if do == "loss":
        return {"bytes": 36.0 * px, "flops": 3.0 * px * (8 * 22 * 2 + 40)}
    if do == "targets":
        f = progressive.downsample_factor(1000)
        return {"bytes": 4.0 * 3 * px * (3 + 1 / f ** 2), "flops": 3.0 * px * (2 + 2 * 2 * 9)}
    proj = nrec * (120.0 + 6.0 * (case["deg"] + 1) ** 2)
    if do == "view":
        return {"bytes": 4.0 * (par * n + 3 * px), "flops": proj + 210.0 * px}
    if do == "lists":
        return {"bytes": 4.0 * par * n + nrec * 56.0, "flops": proj}
    if do == "score":
        return {"bytes": 4.0 * (par + 2) * n, "flops": proj + 140.0 * px}
    return {"bytes": 4.0 * (2 * par * n + 6 * px), "flops": 4.0 * proj + 730.0 * px}


# ---------------------------------------------------------------------------
# the same in 64 bits, from plain torch

MAX_BLOCKS = {"view": 2500, "step": 900, "autograd": 900}  # 32 x 32 pixel blocks done in seconds


def _sh_basis(d):
    """Real spherical harmonics 1..15 (Condon-Shortley sign kept), k = l^2 + l + m, at unit d [3, n]."""
    x, y, z = d
    pi = math.pi
    c1 = math.sqrt(3 / (4 * pi))
    a2, b2, c2 = math.sqrt(15 / pi) / 2, math.sqrt(5 / pi) / 4, math.sqrt(15 / pi) / 4
    a3, b3, c3 = math.sqrt(35 / (2 * pi)) / 4, math.sqrt(105 / pi) / 2, math.sqrt(21 / (2 * pi)) / 4
    d3, e3 = math.sqrt(7 / pi) / 4, math.sqrt(105 / pi) / 4
    return [-c1 * y, c1 * z, -c1 * x,
            a2 * x * y, -a2 * y * z, b2 * (2 * z * z - x * x - y * y), -a2 * x * z, c2 * (x * x - y * y),
            -a3 * y * (3 * x * x - y * y), b3 * x * y * z, -c3 * y * (4 * z * z - x * x - y * y),
            d3 * z * (2 * z * z - 3 * x * x - 3 * y * y), -c3 * x * (4 * z * z - x * x - y * y),
            e3 * z * (x * x - y * y), -a3 * x * (x * x - 3 * y * y)]


def _hard(logit):
    """Hard mask with the straight-through gradient."""
    soft = torch.sigmoid(logit)
    return (soft > 0.5).double() + soft - soft.detach()


def _project64(p, cam, o, n, deg):
    """Records of one view: (u, v), conic, opacity, radius, depth, colour, valid."""
    R = torch.from_numpy(np.asarray(cam.R, np.float64)).to(p["means"].device)
    t = torch.from_numpy(np.asarray(cam.t, np.float64)).to(p["means"].device)[:, None]
    m = _hard(p["mask_logits"]) if "mask_logits" in p else torch.ones_like(p["opacity_logits"])
    x, y, z = R @ p["means"] + t
    valid = (m.detach() > 0.5) & (z.detach() > float(np.float32(o.near_plane)))
    zs = torch.where(valid, z, torch.ones_like(z))
    q = p["quats"] / p["quats"].norm(dim=0, keepdim=True)
    w, i, j, k = q
    Rq = torch.stack([torch.stack([1 - 2 * (j * j + k * k), 2 * (i * j - w * k), 2 * (i * k + w * j)]),
                      torch.stack([2 * (i * j + w * k), 1 - 2 * (i * i + k * k), 2 * (j * k - w * i)]),
                      torch.stack([2 * (i * k - w * j), 2 * (j * k + w * i), 1 - 2 * (i * i + j * j)])])
    M = Rq * (torch.exp(p["log_scales"]) * m)[None]
    lx, ly = (o.tan_clamp * 0.5 * s / f for s, f in ((cam.width, cam.fx), (cam.height, cam.fy)))
    rx, ry = (x / zs).clamp(-lx, lx), (y / zs).clamp(-ly, ly)
    Ta = cam.fx / zs * R[0][:, None] - cam.fx * rx / zs * R[2][:, None]
    Tb = cam.fy / zs * R[1][:, None] - cam.fy * ry / zs * R[2][:, None]
    ma, mb = (Ta[:, None] * M).sum(0), (Tb[:, None] * M).sum(0)
    s = float(np.float32(o.lowpass))
    if o.lowpass_progressive:
        s = max(s, cam.width * cam.height / (9 * math.pi * n))
    ca, cb, cc = (ma * ma).sum(0) + s, (ma * mb).sum(0), (mb * mb).sum(0) + s
    det = ca * cc - cb * cb
    mid = 0.5 * (ca + cc)
    radius = torch.ceil(3 * (mid + (mid * mid - det).clamp(min=0).sqrt()).sqrt()).detach()
    rgb = p["sh_dc"]
    if deg > 0:
        centre = -(R.T @ t)
        d = p["means"] - centre
        Y = _sh_basis(d / d.norm(dim=0, keepdim=True))
        bands = [_hard(b) for b in p["sh_mask_logits"]] if "sh_mask_logits" in p else [1.0] * 3
        for c in range(1, (deg + 1) ** 2):
            rgb = rgb + bands[int(math.isqrt(c)) - 1] * Y[c - 1] * p["sh_rest"][c - 1]
    return dict(u=cam.fx * x / zs + cam.cx, v=cam.fy * y / zs + cam.cy, A=cc / det, B=-cb / det, C=ca / det,
                o=torch.sigmoid(p["opacity_logits"]) * m, rgb=rgb.clamp(min=0), radius=radius, depth=z, valid=valid)


def _block64(rec, sel, x0, x1, y0, y1):
    """Pixels [x0, x1) x [y0, y1) over the depth-ordered records `sel`: [3, pixels]."""
    dev = rec["u"].device
    py, px = torch.meshgrid(torch.arange(y0, y1, device=dev).double() + 0.5,
                            torch.arange(x0, x1, device=dev).double() + 0.5, indexing="ij")
    px, py = px.reshape(-1), py.reshape(-1)
    if sel.numel() == 0:
        return torch.zeros(3, px.numel(), dtype=torch.float64, device=dev)
    r = {k: rec[k][..., sel] for k in ("u", "v", "A", "B", "C", "o", "rgb", "radius")}
    dx, dy = px[None] - r["u"][:, None], py[None] - r["v"][:, None]
    G = torch.exp(-0.5 * (r["A"][:, None] * dx * dx + r["C"][:, None] * dy * dy) - r["B"][:, None] * dx * dy)
    alpha = (r["o"][:, None] * G).clamp(max=float(np.float32(0.99)))
    rad = r["radius"][:, None]
    keep = (dx.detach().abs() <= rad) & (dy.detach().abs() <= rad) & (alpha.detach() >= float(np.float32(1 / 255)))
    alpha = torch.where(keep, alpha, torch.zeros_like(alpha))
    T = torch.cumprod(1 - alpha, 0)
    alive = T.detach() >= float(np.float32(1e-4))  # T only falls: what comes after a stop is stopped too
    T0 = torch.cat([torch.ones_like(T[:1]), T[:-1]], 0)
    w = torch.where(alive, alpha * T0, torch.zeros_like(alpha))
    return r["rgb"] @ w


def _render64(rec, cam, dL=None):
    """The view's image [3, H, W], or (dL given) the gradients of sum(dL * image) left in the records."""
    W, H, B = cam.width, cam.height, 32
    order = torch.argsort(torch.where(rec["valid"], rec["depth"].detach(), torch.full_like(rec["depth"], math.inf)),
                          stable=True)[: int(rec["valid"].sum())]
    u, v, r = rec["u"].detach()[order], rec["v"].detach()[order], rec["radius"][order]
    img = torch.zeros(3, H, W, dtype=torch.float64, device=u.device)
    for y0 in range(0, H, B):
        y1 = min(y0 + B, H)
        row = order[(v + r >= y0) & (v - r <= y1)]
        ur, rr = rec["u"].detach()[row], rec["radius"][row]
        for x0 in range(0, W, B):
            x1 = min(x0 + B, W)
            sel = row[(ur + rr >= x0) & (ur - rr <= x1)]
            out = _block64(rec, sel, x0, x1, y0, y1)
            img[:, y0:y1, x0:x1] = out.detach().view(3, y1 - y0, x1 - x0)
            if dL is not None and sel.numel():
                (out * dL[:, y0:y1, x0:x1].reshape(3, -1)).sum().backward()
    return img


def _window(a, r=5, sigma=1.5):
    """Separable Gaussian window with zero padding over the last two axes."""
    g = torch.exp(-torch.arange(-r, r + 1).double() ** 2 / (2 * sigma ** 2)).to(a.device)
    g = g / g.sum()
    for dim in (-1, -2):
        pad = [r, r, 0, 0] if dim == -1 else [0, 0, r, r]
        b = torch.nn.functional.pad(a, pad)
        a = sum(g[k] * b.narrow(dim, k, a.shape[dim]) for k in range(2 * r + 1))
    return a


def _loss64(images, target, case):
    """(per-view losses and their mean, the gradient) of L1 + D-SSIM."""
    losses, grads, off = [], [], 0
    for (w, h), img in zip(_sizes(case), images):
        x = img.detach().reshape(3, h, w).requires_grad_(True)
        y = target[off:off + 3 * w * h].double().view(3, h, w)
        off += 3 * w * h
        mx, my = _window(x), _window(y)
        sxx, syy, sxy = _window(x * x) - mx * mx, _window(y * y) - my * my, _window(x * y) - mx * my
        ssim = (2 * mx * my + 1e-4) * (2 * sxy + 9e-4) / ((mx * mx + my * my + 1e-4) * (sxx + syy + 9e-4))
        loss = (1 - LAMBDA_SSIM) * (x - y).abs().mean() + LAMBDA_SSIM * (1 - ssim.mean())
        grads.append(torch.autograd.grad(loss / len(images), x)[0].reshape(-1))
        losses.append(loss.detach())
    losses.append(sum(losses) / len(losses))
    return torch.stack(losses), torch.cat(grads)


def _resize64(img, W, H, Wo, Ho):
    def overlap(n, m):
        a = torch.arange(m, device=img.device).double()[:, None] * n / m
        i = torch.arange(n, device=img.device).double()[None]
        return (torch.minimum(a + n / m, i + 1) - torch.maximum(a, i)).clamp(min=0) * m / n
    return overlap(H, Ho) @ img @ overlap(W, Wo).T


def _blur64(img, k, sigma):
    r = k // 2
    g = torch.exp(-torch.arange(-r, r + 1).double() ** 2 / (2 * sigma ** 2)).to(img.device)
    g = g / g.sum()
    for dim in (-1, -2):
        n = img.shape[dim]
        i = torch.arange(-r, n + r, device=img.device).abs()
        i = torch.where(i >= n, 2 * (n - 1) - i, i)
        b = img.index_select(img.dim() + dim, i)
        img = sum(g[j] * b.narrow(dim, j, n) for j in range(k))
    return img


def exact(case, seed):
    do = case["do"]
    if do == "loss":
        loss, grad = _loss64([p.double() for p in _planes(case, seed).split([3 * w * h for w, h in _sizes(case)])],
                             _planes(case, seed + 500_000), case)
        return dict(loss=loss, grad=grad)
    cams, o, n = _cams(case), _opts(case), case["n"]
    if do == "targets":
        img, small, blurred = _planes(case, seed).double(), [], []
        to = progressive.scaled_cameras(cams, progressive.downsample_factor(1000))
        k, sigma = progressive.blur_kernel(1000)
        for (w, h), c, part in zip(_sizes(case), to, img.split([3 * w * h for w, h in _sizes(case)])):
            small.append(_resize64(part.view(3, h, w), w, h, c.width, c.height).reshape(-1))
            blurred.append(_blur64(part.view(3, h, w), k, sigma).reshape(-1))
        return dict(small=torch.cat(small), blurred=torch.cat(blurred))
    p = {k: v.double() for k, v in _params(case, seed).items()}
    if do == "lists":
        if n * len(cams) > 10_000_000:
            return None
        rows = []
        for cam in cams:
            r = _project64(p, cam, o, n, case["deg"])
            rgb = r["rgb"].expand(3, n)
            m = torch.stack([r["u"], r["v"], r["A"], r["B"], r["C"], r["o"], r["radius"], r["depth"], *rgb,
                             torch.ones_like(r["u"])], 1)
            rows.append(torch.where(r["valid"][:, None], m, torch.zeros_like(m)))
        return dict(splats=torch.cat(rows), tiles_touched=None, offsets=None, ids=None, pair_index=None, ranges=None,
                    count=None)
    blocks = sum(-(-w // 32) * -(-h // 32) for w, h in _sizes(case))
    if do not in MAX_BLOCKS or blocks > MAX_BLOCKS[do] or n * len(cams) > 2_000_000:
        return None
    if do == "view":
        with torch.no_grad():
            return dict(image=torch.cat([_render64(_project64(p, c, o, n, case["deg"]), c).reshape(-1) for c in cams]))
    p = {k: v.requires_grad_(True) for k, v in p.items()}
    planes = _planes(case, seed)
    with torch.no_grad():
        images = [_render64(_project64(p, c, o, n, case["deg"]), c) for c in cams]
    out, off, dLs = dict(image=torch.cat([i.reshape(-1) for i in images])), 0, []
    if do == "step" and case["loss"] == "l1_dssim":
        out["loss"], g = _loss64(images, planes, case)
        dLs = list(g.split([3 * w * h for w, h in _sizes(case)]))
    for img in images:
        t = planes[off:off + img.numel()].double().view_as(img)
        off += img.numel()
        if do == "autograd":
            dLs.append(t)
        elif case["loss"] == "l2":
            dLs.append(2 * (img - t) / (img.numel() * len(images)))
    for cam, img, dL in zip(cams, images, dLs):
        rec = _project64(p, cam, o, n, case["deg"])
        grown = [k for k in ("u", "v", "A", "B", "C", "o", "rgb") if rec[k].requires_grad]
        leaf = dict(rec, **{k: rec[k].detach().requires_grad_(True) for k in grown})
        _render64(leaf, cam, dL.reshape(img.shape))
        live = [k for k in grown if leaf[k].grad is not None]
        if live:
            # records that are not composited get no gradient, whatever their projection is
            gs = [torch.where(rec["valid"], leaf[k].grad, torch.zeros_like(leaf[k].grad)) for k in live]
            torch.autograd.backward([rec[k] for k in live], gs)
    grads = {k: v.grad if v.grad is not None else torch.zeros_like(v) for k, v in p.items()}
    if do == "step" and case["loss"] == "l1_dssim":
        total = torch.zeros(1, dtype=torch.float64, device=_device())
        for name, lam, wts in (("mask_logits", LAMBDA_MASK[0], [1.0]), ("sh_mask_logits", LAMBDA_MASK[1], [3.0, 5.0, 7.0])):
            if name not in p or (name == "sh_mask_logits" and case["deg"] == 0):
                continue
            wts = wts[:case["deg"]] if name == "sh_mask_logits" else wts
            for b, wt in enumerate(wts):
                soft = torch.sigmoid((p[name][b] if name == "sh_mask_logits" else p[name]).detach())
                k = lam * wt / sum(wts) / n
                total += k * soft.sum()
                (grads[name][b] if name == "sh_mask_logits" else grads[name]).add_(k * soft * (1 - soft))
        out["mask_loss"] = total
    if do == "step" and not case["sh_rest"] and "sh_rest" in grads:
        grads["sh_rest"] = torch.zeros_like(grads["sh_rest"])
    out["grads"] = grads
    return out
