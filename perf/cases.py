"""The workloads this library is timed on, through its public entry points.

A case is a dict of plain values. `what` names the call:

  step      ActiveBlockStep.step: one training step of the active block on one
            camera (with `layers`, the collapse of that many cached renders
            into F and B beside it)
  train     the calls BlockDescent.visit makes per step: binning that reads
            the intersection count back, forward, loss gradient, backward
  render    train.render_joint: a whole scene rendered for viewing or scoring
  refresh   CacheRefresher.refresh: a block's cached fp16 renders for `cams`
            cameras, down to pinned host memory
  collapse  api.composite_cache: cached renders folded into F and B
  adam      api.adam_step on a block's five parameter groups

and `scene` the distribution of the Gaussians (the recipes of synthetic.py,
drawn on the GPU). `view` is the camera's place on its ellipse, in degrees.
"""
import math

import numpy as np
import torch

from paper_2608_27735_amd import api, synthetic, train
from paper_2608_27735_amd.cache import CacheRefresher
from paper_2608_27735_amd.camera import RasterParams, look_at
from paper_2608_27735_amd.step import ActiveBlockStep

NAMES = ("means", "log_scales", "quats", "opacity_logits", "sh")

# lo, hi of the block; mean and sd of the log-scales; camera ellipse (a, b, z) and target
SCENES = {
    # one 1-unit cell of the 2x2x2 grid, camera at distance 3
    "cell": dict(lo=(-1, -1, -1), hi=(0, 0, 0), ls=math.log(0.03), sd=0.3, cam=(2.78, 2.78, 1.11), at=(0, 0, 0)),
    # one cell of the ring scene's 4x4x4 grid: a blob in it
    "ring": dict(lo=(-0.5, -0.5, -0.5), hi=(0, 0, 0), ls=math.log(0.03), sd=0.3, cam=(2.82, 2.82, 1.03), at=(0, 0, 0), blobs=2, blob_sd=0.08),
    # the whole ring scene
    "rings": dict(lo=(-1, -1, -1), hi=(1, 1, 1), ls=math.log(0.03), sd=0.3, cam=(2.82, 2.82, 1.03), at=(0, 0, 0), blobs=32, blob_sd=0.08),
    # a small scene of mixed sizes, uniform in a cube
    "cube": dict(lo=(-1, -1, -1), hi=(1, 1, 1), ls=math.log(0.05), sd=0.6, cam=(2.8, 2.8, 1.1), at=(0, 0, 0)),
    # the 5-unit active cell, uniform; heavy: a long tail of large Gaussians
    "block": dict(lo=(-2.5, -2.5, 0), hi=(2.5, 2.5, 5), ls=math.log(0.25), sd=0.5, cam=(20, 16, 8), at=(0, 0, 2)),
    "heavy": dict(lo=(-2.5, -2.5, 0), hi=(2.5, 2.5, 5), ls=math.log(0.25), sd=1.0, cam=(20, 16, 8), at=(0, 0, 2)),
    # the mid-scale cell: 40% on the ground, 60% in blobs
    "mid": dict(lo=(-5, -5, 0), hi=(0, 0, 3), ls=math.log(0.2), sd=0.5, cam=(16, 12, 5), at=(0, 0, 1.5), blobs=8, blob_sd=0.5, ground=0.4),
    # tiny Gaussians seen from far
    "stress": dict(lo=(-5, -5, 0), hi=(0, 0, 5), ls=math.log(0.08), sd=0.5, cam=(30, 24, 12), at=(0, 0, 2)),
}


def listed():
    return [
        # the smallest active cell: a step is a handful of short launches, thousands of which make an epoch
        dict(name="cell_128", what="step", scene="cell", n=512, w=128, h=128, sh=0, view=107.0),
        # a small ragged frame: neither side a multiple of the tile, an odd count
        dict(name="ragged_203x117", what="step", scene="cube", n=3001, w=203, h=117, sh=2, view=31.0),
        # a small block in the training loop, which reads the intersection count back every step
        dict(name="ring_train", what="train", scene="ring", n=1024, w=512, h=512, sh=3, view=45.0),
        # a whole small scene rendered for scoring (forward only)
        dict(name="rings_render", what="render", scene="rings", n=65536, w=512, h=512, sh=3, view=45.0),
        # an ordinary active block of a mid-scale scene
        dict(name="mid_300k", what="step", scene="mid", n=300_000, w=1297, h=840, sh=3, view=0.0),
        # the same with visibility-aware skipping: dense front layers, thresholded collapse, early stop
        dict(name="mid_300k_hidden", what="step", scene="mid", n=300_000, w=1297, h=840, sh=3, view=90.0, layers=31, front=12, hide=True),
        # the large active block with the collapse of its 99 frozen neighbours' renders: the headline step
        dict(name="block_1m", what="step", scene="block", n=1_000_000, w=1297, h=840, sh=3, view=0.0, layers=99, front=40),
        # the same block with a heavy tail of large Gaussians at 1080p: the longest lists
        dict(name="heavy_1m_1080p", what="step", scene="heavy", n=1_000_000, w=1920, h=1080, sh=3, view=0.0),
        # many tiny Gaussians on a large frame: bound by what happens per Gaussian
        dict(name="stress_4m_1440p", what="step", scene="stress", n=4_000_000, w=2560, h=1440, sh=3, view=0.0),
        # after a block's steps its cached renders are redrawn for every camera that sees it
        dict(name="refresh_300k", what="refresh", scene="mid", n=300_000, w=1297, h=840, sh=3, view=0.0, cams=4),
        # a camera's F and B when a block becomes active: whole-frame layers
        dict(name="collapse_31_1080p", what="collapse", w=1920, h=1080, layers=31, front=13),
        # the optimizer on a large block
        dict(name="adam_1m", what="adam", n=1_000_000, sh=3),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    what = rng.choice(["step", "step", "step", "train", "render", "refresh", "collapse", "adam"])
    if what == "adam":
        return dict(what="adam", n=_log(rng, 300, 1_500_000), sh=rng.randint(0, 3))
    w = _log(rng, 64, 1920)
    h = max(17, min(1440, int(w * rng.uniform(0.5, 1.1))))
    if what == "collapse":
        k = rng.randint(2, 100)
        return dict(what="collapse", w=w, h=h, layers=k, front=rng.randint(0, k), boxes=rng.random() < 0.5, hide=rng.random() < 0.3)
    scene = rng.choice(["cell", "ring", "cube", "block", "mid", "stress"] if what != "render" else ["rings", "block", "mid"])
    # the small cells hold few Gaussians, the large blocks up to a million
    n = _log(rng, 200, 20_000) if scene in ("cell", "ring", "cube") else _log(rng, 2_000, 1_000_000)
    c = dict(what=what, scene=scene, n=n, w=w, h=h, sh=rng.randint(0, 3), view=round(rng.uniform(0, 360), 1))
    if what == "refresh":
        c["cams"] = rng.randint(1, 5)
    if what == "step" and rng.random() < 0.5:
        c["layers"] = rng.randint(2, 60)
        c["front"] = rng.randint(0, c["layers"])
        c["hide"] = rng.random() < 0.3
    return c


# ------------------------------------------------------------------ inputs

def _dev():
    return torch.device("cuda", torch.cuda.current_device())


def _camera(c, k=0):
    s = SCENES[c["scene"]]
    a = math.radians(c["view"] + 7.2 * k)
    x, y, z = s["cam"]
    return look_at((x * math.cos(a), y * math.sin(a), z), s["at"], c["w"], c["h"])


def _prm(c):
    return RasterParams(sh_degree=c["sh"], fb_stop=bool(c.get("hide", False)))


def _scene(c, seed):
    """The block's parameters (synthetic.gaussians' distributions)."""
    s, n, dev = SCENES[c["scene"]], c["n"], _dev()
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    rand = lambda *shape: torch.rand(shape, generator=g, device=dev)
    randn = lambda *shape: torch.randn(shape, generator=g, device=dev)
    lo = torch.tensor(s["lo"], dtype=torch.float32, device=dev)
    hi = torch.tensor(s["hi"], dtype=torch.float32, device=dev)
    means = lo + (hi - lo) * rand(n, 3)
    ground = int(s.get("ground", 0.0) * n)
    if s.get("blobs"):
        centres = lo + (hi - lo) * rand(s["blobs"], 3)
        comp = torch.randint(s["blobs"], (n - ground,), generator=g, device=dev)
        blob = centres[comp] + s["blob_sd"] * randn(n - ground, 3)
        means[ground:] = torch.minimum(torch.maximum(blob, lo), hi - 1e-6)
    means[:ground, 2] = 0.1 * rand(ground)
    q = randn(n, 4)
    nc = (c["sh"] + 1) ** 2
    sh = 0.1 * randn(n, nc, 3)
    sh[:, 0] = math.sqrt(math.pi) * (2 * rand(n, 3) - 1)
    return dict(means=means.contiguous(), log_scales=s["ls"] + s["sd"] * randn(n, 3),
                quats=q / q.norm(dim=1, keepdim=True), opacity_logits=randn(n), sh=sh)


def _layer(g, h, w, amax, cover):
    """One premultiplied RGBA image: noise over a rectangle of `cover` of the frame."""
    dev = _dev()
    hh, ww = max(1, int(h * math.sqrt(cover))), max(1, int(w * math.sqrt(cover)))
    at = torch.rand(2, generator=g, device=dev).tolist()
    y, x = int(at[0] * (h - hh + 1)), int(at[1] * (w - ww + 1))
    out = torch.zeros((h, w, 4), device=dev)
    a = amax * torch.rand((hh, ww, 1), generator=g, device=dev)
    out[y:y + hh, x:x + ww, :3] = a * torch.rand((hh, ww, 3), generator=g, device=dev)
    out[y:y + hh, x:x + ww, 3:] = a
    return out


def _images(c, seed):
    """F, B (or cached layers with their boxes and order) and the target image.

    The target is black and white: no pixel's L1 difference is near zero,
    where its gradient's sign would hang on the last bit of the render."""
    dev, h, w = _dev(), c["h"], c["w"]
    g = torch.Generator(device=dev)
    g.manual_seed(seed + 1_000_003)
    d = dict(target=(torch.rand((h, w, 3), generator=g, device=dev) < 0.5).float())
    if c.get("layers"):
        cover = 1.0 if c["what"] == "collapse" and not c.get("boxes") else 0.35
        d["layers"], d["rects"] = synthetic.cached_images_device(c["layers"], h, w, seed + 5, dev, coverage=cover, with_rects=True)
        if c.get("hide"):
            # the first layers are dense walls close to the camera
            walls = min(c["layers"], max(1, c["front"] // 4))
            d["layers"][:walls, :, : w // 2, 3] = 0.97
            d["rects"][:walls] = torch.tensor([0, 0, w, h], dtype=torch.int32, device=dev)
        if cover == 1.0:
            d["rects"] = None
        p = torch.randperm(c["layers"], generator=g, device=dev).tolist()
        d["order"] = sorted(range(c["layers"])) if c.get("hide") else p
        d["F"], d["B"] = (torch.empty((h, w, 4), device=dev) for _ in range(2))
    else:
        d["F"], d["B"] = _layer(g, h, w, 0.6, 0.4), _layer(g, h, w, 0.95, 0.7)
    return d


def _stop_t(c):
    return 1e-4 if c.get("hide") else 0.0


def _adam_state(c, seed):
    dev = _dev()
    g = torch.Generator(device=dev)
    g.manual_seed(seed)
    nc = (c["sh"] + 1) ** 2
    shapes = dict(means=(c["n"], 3), log_scales=(c["n"], 3), quats=(c["n"], 4), opacity_logits=(c["n"],), sh=(c["n"], nc, 3))
    randn = lambda s: torch.randn(s, generator=g, device=dev)
    p = {k: randn(s) for k, s in shapes.items()}
    gr = {k: 1e-4 * randn(s) for k, s in shapes.items()}
    m = {k: 1e-5 * randn(s) for k, s in shapes.items()}
    v = {k: 1e-8 * randn(s).square() for k, s in shapes.items()}
    return p, gr, m, v


def prepare(case, seed):
    c = dict(case)
    s = dict(case=c)
    if c["what"] == "adam":
        s["adam"] = _adam_state(c, seed)
        return s
    if c["what"] == "collapse":
        s.update(_images(c, seed))
        return s
    s["params"], s["prm"] = _scene(c, seed), _prm(c)
    if c["what"] == "render":
        s["cam"] = _camera(c)
    elif c["what"] == "refresh":
        s["cams"] = [_camera(c, k) for k in range(c["cams"])]
        s["refresher"] = CacheRefresher(s["prm"], s["params"], c["w"], c["h"])
        s["host"] = torch.empty((c["cams"], c["h"], c["w"], 4), dtype=torch.float16, pin_memory=True)
        s["boxes"] = torch.zeros((c["cams"], 4), dtype=torch.int32, device=_dev())
    else:
        s.update(_images(c, seed))
        s["step"] = ActiveBlockStep(_camera(c), s["prm"], s["params"])
    return s


# -------------------------------------------------------------------- calls

def run(s):
    c = s["case"]
    what = c["what"]
    if what == "adam":
        p, g, m, v = s["adam"]
        api.adam_step(p, g, m, v, train.DEFAULT_LR, 10)
        return dict(param=p, exp_avg=m, exp_avg_sq=v)
    if what == "collapse":
        return api.composite_cache(s["layers"], s["order"], c["front"], F=s["F"], B=s["B"], rects=s["rects"], stop_t=_stop_t(c))
    if what == "render":
        return train.render_joint(s["cam"], s["prm"], s["params"])
    if what == "refresh":
        s["refresher"].refresh(s["cams"], list(s["host"]), s["boxes"])
        return s["host"], s["boxes"]
    st, F, B = s["step"], s["F"], s["B"]
    if what == "train":
        st.project_and_bin(sync=True)
        st.forward(F, B)
        st.loss_grad(s["target"])
        st.backward(st.dL_dout, F, B)
    elif c.get("layers"):
        st.step(s["target"], F, B, collapse=lambda: api.composite_cache(
            s["layers"], s["order"], c["front"], F=F, B=B, rects=s["rects"], stop_t=_stop_t(c), beside=True))
    else:
        st.step(s["target"], F, B)
    out = dict(out=st.fwd["out"], final_T=st.fwd["final_T"], grads=st.grads)
    if c.get("layers"):
        out["F"], out["B"] = F, B
    return out


# ------------------------------------------------------------- cost and bars

def work(case):
    c = case
    nc = (c.get("sh", 0) + 1) ** 2
    floats = 11 + 3 * nc  # parameters of one Gaussian
    if c["what"] == "adam":
        return dict(bytes=28 * c["n"] * floats, flops=12 * c["n"] * floats)
    px = c["w"] * c["h"]
    layer = 0
    if c.get("layers"):
        cover = 1.0 if c["what"] == "collapse" and not c.get("boxes") else 0.35
        layer = c["layers"] * px * cover
    if c["what"] == "collapse":
        return dict(bytes=8 * layer + 32 * px, flops=8 * layer)
    # a pixel blends some tens of entries before it saturates (about 65 on the
    # 1M block), at about 20 operations forward and 60 backward each
    blends = 40 * px
    if c["what"] == "render":
        return dict(bytes=4 * floats * c["n"] + 16 * px, flops=300 * c["n"] + 20 * blends)
    if c["what"] == "refresh":
        return dict(bytes=c["cams"] * (4 * floats * c["n"] + 8 * px), flops=c["cams"] * (300 * c["n"] + 20 * blends))
    return dict(bytes=8 * floats * c["n"] + (32 + 12 + 20) * px + 8 * layer, flops=900 * c["n"] + 80 * blends + 8 * layer)


def tolerance(case):
    """About four times what separates the outputs from exact()'s."""
    what = case["what"]
    if what == "adam":
        return dict(rel=2e-7, max=1e-5)
    if case.get("hide"):
        # a layer or an entry is left out once less than 1e-4 of it shows, and
        # 1 - alpha that small holds three digits: some pixels fall either way
        return dict(rel=5e-3, max=0.9)
    if what == "collapse":
        return dict(rel=4e-7, max=1e-5)
    if what == "refresh":
        return dict(rel=8e-4, max=0.05, differ=0.01)  # binary16 images
    # an entry at alpha_min or a pixel at t_min may go either way in the last
    # bit, which moves that pixel, and the gradients of what it blends
    if what == "render":
        return dict(rel=5e-5, max=0.05)
    return dict(rel=2e-3, max=0.9)


# --------------------------------------------------- the same in 64 bits

def _sh_basis(d):
    x, y, z = d.unbind(1)
    xx, yy, zz = x * x, y * y, z * z
    r = math.sqrt
    pi = math.pi
    return torch.stack([
        torch.full_like(x, r(1 / (4 * pi))),
        r(3 / (4 * pi)) * y, r(3 / (4 * pi)) * z, r(3 / (4 * pi)) * x,
        r(15 / (4 * pi)) * x * y, r(15 / (4 * pi)) * y * z, r(5 / (16 * pi)) * (2 * zz - xx - yy),
        r(15 / (4 * pi)) * x * z, r(15 / (16 * pi)) * (xx - yy),
        r(35 / (32 * pi)) * y * (3 * xx - yy), r(105 / (4 * pi)) * x * y * z,
        r(21 / (32 * pi)) * y * (4 * zz - xx - yy), r(7 / (16 * pi)) * z * (2 * zz - 3 * xx - 3 * yy),
        r(21 / (32 * pi)) * x * (4 * zz - xx - yy), r(105 / (16 * pi)) * z * (xx - yy),
        r(35 / (32 * pi)) * x * (xx - 3 * yy)], dim=1)


def _project64(cam, prm, p):
    """Screen-space values of every Gaussian in float64 (differentiable), the
    fp32 depth that orders the lists, and each box as tile coordinates."""
    dev = _dev()
    t64 = lambda a: torch.tensor(np.asarray(a, np.float64), device=dev)
    R, t, pos = t64(cam.R).reshape(3, 3), t64(cam.t), t64(cam.campos)
    x = p["means"] @ R.T + t
    tz = x[:, 2]
    tx, ty = x[:, 0] / tz, x[:, 1] / tz
    u, v = cam.fx * tx + cam.cx, cam.fy * ty + cam.cy
    lx, ly = prm.guard * cam.width / (2 * cam.fx), prm.guard * cam.height / (2 * cam.fy)
    cxn, cyn = tx.clamp(-lx, lx), ty.clamp(-ly, ly)
    zero = torch.zeros_like(tz)
    J = torch.stack([cam.fx / tz, zero, -cam.fx * cxn / tz, zero, cam.fy / tz, -cam.fy * cyn / tz], dim=1).reshape(-1, 2, 3)
    q = p["quats"] / p["quats"].norm(dim=1, keepdim=True)
    w, i, j, k = q.unbind(1)
    rot = torch.stack([1 - 2 * (j * j + k * k), 2 * (i * j - w * k), 2 * (i * k + w * j),
                       2 * (i * j + w * k), 1 - 2 * (i * i + k * k), 2 * (j * k - w * i),
                       2 * (i * k - w * j), 2 * (j * k + w * i), 1 - 2 * (i * i + j * j)], dim=1).reshape(-1, 3, 3)
    # J R rot diag(s): 2x3, its square the covariance
    A = ((J[:, :, None, :] * R.T[None, None]).sum(-1)[:, :, :, None] * rot[:, None]).sum(2) * p["log_scales"].exp()[:, None, :]
    ca = (A[:, 0] ** 2).sum(1) + prm.eps2d
    cb = (A[:, 0] * A[:, 1]).sum(1)
    cc = (A[:, 1] ** 2).sum(1) + prm.eps2d
    det = ca * cc - cb * cb
    conic = torch.stack([cc / det, -cb / det, ca / det], dim=1)
    o = torch.sigmoid(p["opacity_logits"])
    d = p["means"] - pos
    nc = (prm.sh_degree + 1) ** 2
    Y = _sh_basis(d / d.norm(dim=1, keepdim=True))[:, :nc]
    rgb = ((Y[:, :, None] * p["sh"]).sum(1) + 0.5).clamp_min(0.0)
    val = torch.cat([u[:, None], v[:, None], conic, o[:, None], rgb], dim=1)
    with torch.no_grad():
        r32 = [np.float32(a) for a in np.asarray(cam.R, np.float32).reshape(-1)]
        m32 = p["means"].float()
        # fp32, products and sums each rounded, left to right: the sort key
        depth = (float(r32[6]) * m32[:, 0] + float(r32[7]) * m32[:, 1]) + float(r32[8]) * m32[:, 2] + float(np.float32(cam.t[2]))
        mid = 0.5 * (ca + cc)
        rad = prm.radius_sigmas * (mid + (mid * mid - det).clamp_min(0).sqrt()).sqrt()
        man, ex = math.frexp(float(np.float32(prm.alpha_min)))
        L = 1.001 * 2 * ((1 - ex) * math.log(2) + p["opacity_logits"].clamp_max(0)) + 0.001
        ew, eh = torch.minimum(rad, (L.clamp_min(0) * ca).sqrt()), torch.minimum(rad, (L.clamp_min(0) * cc).sqrt())
        ntx, nty = (cam.width + 15) // 16, (cam.height + 15) // 16
        x0, x1 = ((u - ew) / 16).floor().clamp_min(0), ((u + ew) / 16).floor().clamp_max(ntx - 1)
        y0, y1 = ((v - eh) / 16).floor().clamp_min(0), ((v + eh) / 16).floor().clamp_max(nty - 1)
        ok = (tz > cam.near) & (det > 0) & (L > 0) & (x0 <= x1) & (y0 <= y1)
        box = torch.stack([x0, y0, x1, y1], dim=1)
        box[~ok] = 0
        box = box.long()
        count = torch.where(ok, (box[:, 2] - box[:, 0] + 1) * (box[:, 3] - box[:, 1] + 1), torch.zeros_like(box[:, 0]))
    return val, depth, box, count


def _lists(cam, depth, box, count):
    """Gaussians of each tile, front to back: (list, start, length)."""
    ntx, nty = (cam.width + 15) // 16, (cam.height + 15) // 16
    order = torch.sort(depth, stable=True).indices
    cnt = count[order]
    g = torch.repeat_interleave(order, cnt)
    rank = torch.arange(g.numel(), device=g.device) - torch.repeat_interleave(cnt.cumsum(0) - cnt, cnt)
    bw = (box[:, 2] - box[:, 0] + 1)[g]
    tile = ((box[:, 1][g] + rank // bw) * ntx + box[:, 0][g] + rank % bw).to(torch.int32)
    del rank, bw
    tile, at = torch.sort(tile, stable=True)
    length = torch.bincount(tile, minlength=ntx * nty)
    return g[at], length.cumsum(0) - length, length


def _over(f, b):
    return f + (1 - f[..., 3:]) * b


def _blend64(cam, prm, val, lists, F, B, dL=None, chunk=128, batch=64):
    """out and final_T in float64 and, with dL (a function of out), the
    gradient with respect to `val`."""
    g, start, length = lists
    dev, H, W = val.device, cam.height, cam.width
    ntx, nty = (W + 15) // 16, (H + 15) // 16
    amin, amax, tmin = (float(np.float32(a)) for a in (prm.alpha_min, prm.alpha_max, prm.t_min))
    pad = lambda im: torch.nn.functional.pad(im, (0, 0, 0, ntx * 16 - W, 0, nty * 16 - H))
    tiled = lambda im: pad(im).reshape(nty, 16, ntx, 16, -1).permute(0, 2, 1, 3, 4).reshape(nty * ntx, 256, -1)
    back = lambda a: a.reshape(nty, ntx, 16, 16, -1).permute(0, 2, 1, 3, 4).reshape(nty * 16, ntx * 16, -1)[:H, :W]
    Ft, Bt = tiled(F), tiled(B)
    vis = 1 - Ft[..., 3] if prm.fb_stop else torch.ones_like(Ft[..., 3])
    C = torch.zeros((nty * ntx, 256, 3), dtype=torch.float64, device=dev)
    T = torch.ones((nty * ntx, 256), dtype=torch.float64, device=dev)
    px = torch.arange(256, device=dev)
    by_len = torch.argsort(length, descending=True)

    def alphas(tiles, at):
        """alpha of the chunk's entries at the tiles' pixels, and what made it."""
        pos = at + torch.arange(chunk, device=dev)
        have = pos[None] < length[tiles][:, None]
        idx = g[(start[tiles][:, None] + pos[None]).clamp_max(max(g.numel() - 1, 0))]
        s = val[idx]
        x = ((tiles % ntx) * 16)[:, None] + px % 16 + 0.5
        y = ((tiles // ntx) * 16)[:, None] + px // 16 + 0.5
        dx, dy = x[:, :, None] - s[:, None, :, 0], y[:, :, None] - s[:, None, :, 1]
        e = (-0.5 * (s[:, None, :, 2] * dx * dx + s[:, None, :, 4] * dy * dy) - s[:, None, :, 3] * dx * dy).exp()
        raw = s[:, None, :, 5] * e
        a = raw.clamp_max(amax)
        return idx, s, dx, dy, raw, torch.where((raw >= amin) & have[:, None, :], a, torch.zeros_like(a))

    def walk(a, T0, tiles):
        """Transmittance before each entry, and whether the pixel blends it."""
        after = T0[..., None] * (1 - a).cumprod(-1)
        lives = after * vis[tiles][..., None] >= tmin
        before = torch.cat([T0[..., None], after[..., :-1]], -1)
        hit = (a > 0) & lives
        # transmittance kept: of the last entry blended
        kept = torch.where(lives, after, torch.full_like(after, 2.0)).amin(-1)
        return before, hit, torch.where(kept > 1.5, T0, kept), lives[..., -1]

    def sweep(body):
        for b0 in range(0, by_len.numel(), batch):
            tiles = by_len[b0:b0 + batch]
            Tc = torch.ones((tiles.numel(), 256), dtype=torch.float64, device=dev)
            alive = vis[tiles] >= tmin
            at = 0
            while tiles.numel():
                keep = (length[tiles] > at) & alive.any(1)
                if not bool(keep.all()):
                    tiles, Tc, alive = tiles[keep], Tc[keep], alive[keep]
                    continue
                e = alphas(tiles, at)
                before, hit, Tn, lives = walk(e[5], Tc, tiles)
                hit = hit & alive[..., None]
                body(tiles, e, before, hit)
                Tc = torch.where(alive, Tn, Tc)
                T[tiles] = Tc
                alive = alive & lives
                at += chunk

    def forward(tiles, e, before, hit):
        wgt = torch.where(hit, e[5] * before, torch.zeros_like(before))
        C[tiles] += wgt @ e[1][:, :, 6:9]

    sweep(forward)
    A = torch.cat([C + T[..., None] * Bt[..., :3], 1 - T[..., None] * (1 - Bt[..., 3:])], -1)
    out = _over(Ft, A)
    out_im, T_im = back(out), back(T[..., None])[..., 0]
    if dL is None:
        return out_im, T_im, None
    G = tiled(dL(out_im)) * (1 - Ft[..., 3:])
    gT = (G[..., :3] * Bt[..., :3]).sum(-1) - G[..., 3] * (1 - Bt[..., 3])
    total = (C * G[..., :3]).sum(-1) + T * gT
    seen = torch.zeros_like(total)
    dval = torch.zeros_like(val)

    def backward(tiles, e, before, hit):
        idx, s, dx, dy, raw, a = e
        zero = torch.zeros_like(a)
        gc = G[tiles][..., :3]
        wgt = torch.where(hit, a * before, zero)
        cg = gc @ s[:, :, 6:9].transpose(1, 2).contiguous()
        pre = seen[tiles][..., None] + (wgt * cg).cumsum(-1)
        seen[tiles] = pre[..., -1]
        da = torch.where(hit & (raw <= amax), before * cg - (total[tiles][..., None] - pre) / (1 - a), zero)
        dp = da * a  # alpha = raw where the derivative is not cut
        sa, sb, sc = (s[:, None, :, q] for q in (2, 3, 4))
        f = torch.stack([(dp * (sa * dx + sb * dy)).sum(1), (dp * (sc * dy + sb * dx)).sum(1),
                         (-0.5 * dp * dx * dx).sum(1), (-dp * dx * dy).sum(1), (-0.5 * dp * dy * dy).sum(1),
                         (da * raw).sum(1) / s[:, :, 5],
                         *((wgt * gc[..., ch:ch + 1]).sum(1) for ch in range(3))], -1)
        dval.index_add_(0, idx.reshape(-1), f.reshape(-1, 9))

    sweep(backward)
    return out_im, T_im, dval


def _fold64(images, order, n_front, stop_t):
    h, w = images.shape[1:3]
    F = torch.zeros((h, w, 4), dtype=torch.float64, device=images.device)
    B = torch.zeros_like(F)
    for k, j in enumerate(order):
        x = images[j].double()
        if k < n_front:
            on = (1 - F[..., 3:]) >= stop_t
            F = torch.where(on, _over(F, x), F)
        else:
            on = (1 - F[..., 3:]) * (1 - B[..., 3:]) >= stop_t
            B = torch.where(on, _over(B, x), B)
    return F, B


def exact(case, seed):
    c = dict(case)
    what = c["what"]
    if what == "adam":
        p, g, m, v = _adam_state(c, seed)
        b1, b2 = float(np.float32(0.9)), float(np.float32(0.999))
        out = dict(param={}, exp_avg={}, exp_avg_sq={})
        for k in NAMES:
            gd = g[k].double()
            md = b1 * m[k].double() + (1 - b1) * gd
            vd = b2 * v[k].double() + (1 - b2) * gd * gd
            step = train.DEFAULT_LR[k] * (md / (1 - b1 ** 10)) / ((vd / (1 - b2 ** 10)).sqrt() + 1e-15)
            out["param"][k], out["exp_avg"][k], out["exp_avg_sq"][k] = p[k].double() - step, md, vd
        return out
    if what == "collapse":
        d = _images(c, seed)
        return _fold64(d["layers"], d["order"], c["front"], _stop_t(c))
    prm = _prm(c)
    params = {k: v.double().requires_grad_(what in ("step", "train")) for k, v in _scene(c, seed).items()}
    clear = lambda: torch.zeros((c["h"], c["w"], 4), dtype=torch.float64, device=_dev())
    if what in ("render", "refresh"):
        outs = []
        for k in range(c.get("cams", 1)):
            cam = _camera(c, k)
            val, depth, box, count = _project64(cam, prm, params)
            outs.append(_blend64(cam, prm, val, _lists(cam, depth, box, count), clear(), clear())[0])
        return outs[0] if what == "render" else (torch.stack(outs), None)
    d, cam = _images(c, seed), _camera(c)
    if c.get("layers"):
        d["F"], d["B"] = _fold64(d["layers"], d["order"], c["front"], _stop_t(c))
    F, B, target = (d[k].double() for k in ("F", "B", "target"))
    val, depth, box, count = _project64(cam, prm, params)

    def dL(out):
        g = torch.sign(out[..., :3] - target) / (3 * c["w"] * c["h"])
        return torch.cat([g, torch.zeros_like(g[..., :1])], -1)

    out, T, dval = _blend64(cam, prm, val.detach(), _lists(cam, depth, box, count), F, B, dL)
    val.backward(dval)
    res = dict(out=out, final_T=T, grads={k: params[k].grad for k in NAMES})
    if c.get("layers"):
        res["F"], res["B"] = F, B
    return res
