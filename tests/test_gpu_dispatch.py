"""Kernels at the sizes where their paths change: tile edges, remainders,
alignment, the ends of a dispatch rule. Each against the CPU oracle."""
import numpy as np
import pytest
import torch

from oracle import oracle as O
from paper_2608_27735_amd import synthetic as S

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def api():
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    from paper_2608_27735_amd import api as A
    return A


def dev():
    return torch.device("cuda:0")


def say(*a):
    print("[case]", *a, flush=True)


@pytest.mark.parametrize("offset", [0, 1, 4])
@pytest.mark.parametrize("count", [1, 3, 4095, 4096, 4097, 8195])
def test_adam_workgroup_edges(api, count, offset):
    """Counts around the 4,096 elements of a workgroup, aligned and not, beside
    a second group; elements before and after the arrays stay as they were.
    Bars: each moment's rounding on its terms' magnitudes, the update's on its
    own (fp32 evaluation: a few 2^-24 each)."""
    r = S.rng(300 + count + offset)
    say("adam", count, offset)
    f = np.float32
    host = [r.normal(size=count + offset + 8).astype(f) for _ in range(4)]
    host[3] = np.abs(host[3])
    big = [torch.from_numpy(h).to(dev()) for h in host]
    view = [b[offset:offset + count] for b in big]
    other = [torch.ones(5, device=dev()) for _ in range(4)]
    api.adam_step(dict(a=view[0], b=other[0]), dict(a=view[1], b=other[1]),
                  dict(a=view[2], b=other[2]), dict(a=view[3], b=other[3]), 1e-2, 7)
    torch.cuda.synchronize()
    got = [b.cpu().numpy() for b in big]
    keep = np.ones(count + offset + 8, bool)
    keep[offset:offset + count] = False
    for h, g in zip(host, got):
        assert np.array_equal(h[keep], g[keep])
    assert np.array_equal(host[1], got[1])
    t0, g0, m0, v0 = (h[offset:offset + count].astype(np.float64) for h in host)
    b1, b2, lr = float(f(0.9)), float(f(0.999)), float(f(1e-2))
    rt, rm, rv = O.adam(t0, g0, m0, v0, lr, b1, b2, float(f(1e-15)), 7)
    gt, _, gm, gv = (g[offset:offset + count].astype(np.float64) for g in got)
    assert np.all(np.abs(gm - rm) <= 3e-7 * (b1 * np.abs(m0) + (1 - b1) * np.abs(g0)))
    assert np.all(np.abs(gv - rv) <= 3e-7 * (b2 * v0 + (1 - b2) * g0 * g0))
    step = lr / (1 - b1 ** 7) * (b1 * np.abs(m0) + (1 - b1) * np.abs(g0))
    denom = np.sqrt(rv / (1 - b2 ** 7)) + float(f(1e-15))
    assert np.all(np.abs(gt - rt) <= 4e-7 * np.abs(t0) + 2e-6 * step / denom)


@pytest.mark.parametrize("logit", [-4.0, 0.0, 4.0])
@pytest.mark.parametrize("count", [1, 3, 4, 5, 64, 255, 256, 257, 513])
def test_forward_list_lengths(api, count, logit, size=(272, 256)):
    """Lists of 1 to 513 entries in the same few tiles (groups of four, batches
    of 256 and their remainders), faint, saturating within a group, and opaque,
    on a frame of 272 tiles (the general forward; the backward takes lists of 128
    entries or more in rows, shorter ones whole); also t_min = 0 (no stop) and
    an alpha_min that no fp32 alpha falls below. Bars: the parity bars of the
    forward (max abs 1e-5 off knife-edge pixels) and of the gradients (1e-4)."""
    from paper_2608_27735_amd.camera import RasterParams, look_at
    r = S.rng(400 + count)
    cam = look_at((0.0, -3.0, 0.0), (0, 0, 0), *size)
    sc = S.gaussians(r, r.uniform(-0.1, 0.1, (count, 3)), 0, np.log(0.1), 0.3)
    sc["opacity_logits"] = np.full(count, logit, np.float32)
    F, B = S.background_pair(r, cam.height, cam.width)
    dL = S.upstream_grad(r, cam.height, cam.width)
    for kw in (dict(), dict(t_min=0.0), dict(alpha_min=1e-30)):
        prm = RasterParams(sh_degree=0, **kw)
        say("list lengths", count, logit, kw)
        ref = O.step(cam, prm, sc, F=F, B=B, dL_dout=None, rel_margin=1e-4)
        knife = ref["fwd"]["knife"]
        up = np.where(knife[..., None], 0, dL).astype(np.float32)
        ref = O.step(cam, prm, sc, F=F, B=B, dL_dout=up.astype(np.float64), rel_margin=1e-4)
        d = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to(dev())
        params = {k: d(v) for k, v in sc.items()}
        proj = api.project(cam, prm, **params)
        bins = api.bin_sort(cam.width, cam.height, proj)
        length = int((bins["tile_ranges"][:, 1] - bins["tile_ranges"][:, 0]).max())
        assert length == count and bins["n_isect"] <= 65536
        fwd = api.render_fwd(cam, prm, bins, proj, F=d(F), B=d(B))
        grads = api.render_bwd(cam, prm, params, proj, bins, fwd, d(up), F=d(F), B=d(B))
        torch.cuda.synchronize()
        err = np.abs(fwd["out"].cpu().numpy() - ref["fwd"]["out"])[~knife]
        assert err.max() <= 1e-5
        assert np.array_equal(fwd["last"].cpu().numpy().view(np.uint32)[~knife],
                              ref["fwd"]["last"][~knife])
        if prm.t_min == 0.0:
            continue  # 0.5^255 underflows fp32: no backward can recover the walk from final_T
        for k in params:
            g, gr = grads[k].cpu().numpy().astype(np.float64), ref["grads"][k]
            assert np.linalg.norm(g - gr) <= 1e-4 * max(np.linalg.norm(gr), 1e-30), k


@pytest.mark.parametrize("size", [(272, 256), (128, 128)])
def test_backward_upstream_nan_stays_local(api, size):
    """A NaN in the upstream gradient of one pixel reaches only Gaussians whose
    tiles hold that pixel: entries past the end of a group and pixels that blend
    nothing add exact zeros whatever the staged data holds."""
    from paper_2608_27735_amd.camera import RasterParams, look_at
    r = S.rng(500)
    cam = look_at((0.0, -3.0, 0.0), (0, 0, 0), *size)
    sc = S.gaussians(r, r.uniform(-1.0, 1.0, (301, 3)), 0, np.log(0.03), 0.3)
    prm = RasterParams(sh_degree=0)
    say("nan upstream", size)
    d = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to(dev())
    params = {k: d(v) for k, v in sc.items()}
    proj = api.project(cam, prm, **params)
    bins = api.bin_sort(cam.width, cam.height, proj)
    fwd = api.render_fwd(cam, prm, bins, proj)
    dL = S.upstream_grad(r, cam.height, cam.width)
    clean = api.render_bwd(cam, prm, params, proj, bins, fwd, d(dL))
    dL[size[1] // 2, size[0] // 2] = np.nan
    bad = api.render_bwd(cam, prm, params, proj, bins, fwd, d(dL))
    torch.cuda.synchronize()
    ntx = (cam.width + 15) // 16
    tile = (size[1] // 2) // 16 * ntx + (size[0] // 2) // 16
    a, b = bins["tile_ranges"].cpu().numpy()[tile]
    listed = np.zeros(301, bool)
    listed[bins["values"].cpu().numpy()[a:b]] = True
    for k in params:
        g, c = bad[k].cpu().numpy().reshape(301, -1), clean[k].cpu().numpy().reshape(301, -1)
        assert np.isfinite(g[~listed]).all(), k
        # the order of the atomic adds differs between the two calls
        assert np.linalg.norm(g[~listed] - c[~listed]) <= 1e-5 * np.linalg.norm(c), k


@pytest.mark.parametrize("n", [2048, 2049, 4099, 300_001])
def test_binning_without_capacity_counts(api, n):
    """A call with no capacity leaves the intersection count of a full call, empty
    ranges and the identity order, on both sides of the small-block path."""
    from paper_2608_27735_amd.camera import RasterParams, look_at
    r = S.rng(600 + n)
    cam = look_at((0.2, -3.0, 0.9), (0, 0, 0), 203, 117)
    sc = S.gaussians(r, r.uniform(-2, 2, (n, 3)), 0, np.log(0.02), 0.6)
    say("no capacity", n)
    proj = api.project(cam, RasterParams(sh_degree=0),
                       **{k: torch.from_numpy(v).to(dev()) for k, v in sc.items()})
    full = api.bin_sort(cam.width, cam.height, proj)
    got = api.bin_sort(cam.width, cam.height, proj, capacity=0, sync=False)
    assert api.intersections(got["workspace"]) == full["n_isect"]
    assert full["n_isect"] == int(proj["tiles_touched"].sum())
    assert int(got["tile_ranges"].abs().max()) == 0
    assert torch.equal(got["tile_order"].cpu(), torch.arange(len(got["tile_order"]), dtype=torch.int32))


@pytest.mark.parametrize("count", [1, 3, 4, 5, 64, 127, 255, 256, 257, 513])
def test_backward_list_lengths_whole(api, count):
    """The same lists on 1,056 tiles, where the backward takes each tile whole, from
    the queue: groups of four, batches of 256 and their remainders."""
    test_forward_list_lengths(api, count, -4.0, size=(528, 512))


@pytest.mark.parametrize("size", [(272, 256), (505, 499)])
@pytest.mark.parametrize("n", [1500, 40_000])
def test_layout_by_pairs(api, n, size):
    """Frames of 272 and 1,024 tiles whose lists, of 1 to more than 128 entries, hold
    fewer and more pairs than the backward takes long lists in rows for, unsplit,
    split and as a cached render: parity bars against the oracle, and the split and
    unsplit forwards bit-identical."""
    from paper_2608_27735_amd.camera import RasterParams, look_at
    r = S.rng(700 + n)
    cam = look_at((0.1, -3.0, 0.8), (0, 0, 0), *size)
    prm = RasterParams(sh_degree=0)
    sc = S.gaussians(r, r.uniform(-0.6, 0.6, (n, 3)), 0, np.log(0.02), 0.4)
    F, B = S.background_pair(r, cam.height, cam.width)
    ref = O.step(cam, prm, sc, F=F, B=B, rel_margin=1e-4)
    m = len(ref["sorted_values"])
    say("layout by pairs", n, size, m)
    assert (m <= 65536) == (n == 1500)
    length = ref["tile_ranges"][:, 1].astype(np.int64) - ref["tile_ranges"][:, 0]
    if size == (272, 256):
        assert length.max() >= 128 and (length[length > 0] < 128).any()
    knife = ref["fwd"]["knife"]
    dL = np.where(knife[..., None], 0, S.upstream_grad(r, cam.height, cam.width)).astype(np.float32)
    ref = O.step(cam, prm, sc, F=F, B=B, dL_dout=dL.astype(np.float64), rel_margin=1e-4)
    d = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to(dev())
    params = {k: d(v) for k, v in sc.items()}
    proj = api.project(cam, prm, **params)
    bins = api.bin_sort(cam.width, cam.height, proj)
    split = api.make_split(m // 256 + api.n_tiles(*size) + 1, 256)
    outs = []
    for sp in (None, split):
        fwd = api.render_fwd(cam, prm, bins, proj, F=d(F), B=d(B), split=sp)
        grads = api.render_bwd(cam, prm, params, proj, bins, fwd, d(dL), F=d(F), B=d(B), split=sp)
        torch.cuda.synchronize()
        outs.append(fwd)
        err = np.abs(fwd["out"].cpu().numpy() - ref["fwd"]["out"])[~knife]
        assert err.max() <= 1e-5
        assert np.array_equal(fwd["last"].cpu().numpy().view(np.uint32)[~knife],
                              ref["fwd"]["last"][~knife])
        for k in params:
            g, gr = grads[k].cpu().numpy().astype(np.float64), ref["grads"][k]
            assert np.linalg.norm(g - gr) <= 1e-4 * max(np.linalg.norm(gr), 1e-30), (k, sp is None)
    for k in ("out", "final_T", "last"):
        assert torch.equal(outs[0][k], outs[1][k])
    plain = api.render_fwd(cam, prm, bins, proj)["out"]
    assert torch.equal(api.render_cache(cam, prm, bins, proj), plain.half())


@pytest.mark.parametrize("size", [(203, 117), (4096, 128), (128, 4096), (720, 640)])
@pytest.mark.parametrize("n", [1, 1024, 1025, 2049, 4097, 8192, 8193])
def test_binning_small_block_sizes(api, n, size):
    """Blocks on both sides of each size of the one-workgroup sort (1,024 to 8,192
    Gaussians) and of the general path, on frames of 104 tiles, of the widest
    and the highest it takes, and of 1,800, with rectangles from one tile to the
    whole frame: lists, keys, ranges and M bit-exact against the oracle."""
    from paper_2608_27735_amd.camera import RasterParams, look_at
    r = S.rng(800 + n)
    cam = look_at((0.2, -3.0, 0.9), (0, 0, 0), *size)
    sc = S.gaussians(r, r.uniform(-1.5, 1.5, (n, 3)), 0, np.log(0.02), 1.2)
    sc["means"][3::7, 1] -= 4.0  # some behind the camera
    sc["means"][0] = 0.0  # and one in view
    prm = RasterParams(sh_degree=0)
    say("small blocks", n, size)
    pb = O.project_bin(cam, prm, sc["means"], sc["log_scales"], sc["quats"], sc["opacity_logits"])
    keys, values, ranges = O.bin(cam.width, cam.height, pb["depth"], pb["rect"], pb["tiles_touched"])
    proj = api.project(cam, prm, **{k: torch.from_numpy(v).to(dev()) for k, v in sc.items()})
    b = api.bin_sort(cam.width, cam.height, proj, want_keys=True)
    m = b["n_isect"]
    assert m == len(values)
    assert np.array_equal(b["values"][:m].cpu().numpy().view(np.uint32), values)
    assert np.array_equal(b["keys"][:m].cpu().numpy().view(np.uint64), keys)
    assert np.array_equal(b["tile_ranges"].cpu().numpy().view(np.uint32), ranges)


def test_binning_counts_from_several_threads(api):
    """The count is read back through words that calls share: threads on streams
    of their own each get the count of their own block."""
    import threading
    from paper_2608_27735_amd.camera import RasterParams, look_at
    cam = look_at((0.2, -3.0, 0.9), (0, 0, 0), 203, 117)
    projs, wrong = [], []
    for n in (300, 900, 2500, 6000):
        r = S.rng(900 + n)
        sc = S.gaussians(r, r.uniform(-1, 1, (n, 3)), 0, np.log(0.02), 0.6)
        projs.append(api.project(cam, RasterParams(sh_degree=0),
                                 **{k: torch.from_numpy(v).to(dev()) for k, v in sc.items()}))
    want = [int(p["tiles_touched"].sum()) for p in projs]
    say("counts from threads", want)
    torch.cuda.synchronize()

    def work(k):
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(20):
                m = api.bin_sort(cam.width, cam.height, projs[k])["n_isect"]
                if m != want[k]:
                    wrong.append((k, m))

    threads = [threading.Thread(target=work, args=(k,)) for k in range(len(projs))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong
    assert len(set(want)) == len(want)


@pytest.mark.parametrize("size", [(16, 16), (9, 7), (32, 16), (33, 9)])
def test_split_of_a_few_tiles_without_an_order(api, size):
    """A split forward of one, two and three tiles with no tile order: the grid is
    rounded up to eight workgroups, of which those past the last tile do nothing.
    Parity bars against the oracle, for lists longer than a chunk."""
    from paper_2608_27735_amd.camera import RasterParams, look_at
    r = S.rng(1000 + size[0])
    cam = look_at((0.0, -3.0, 0.0), (0, 0, 0), *size, fov_x_deg=20.0)
    prm = RasterParams(sh_degree=0)
    sc = S.gaussians(r, r.uniform(-0.4, 0.4, (900, 3)), 0, np.log(0.05), 0.4)
    sc["opacity_logits"] -= 4.0  # faint, so that the walks cross the chunks
    F, B = S.background_pair(r, cam.height, cam.width)
    say("split without an order", size)
    ref = O.step(cam, prm, sc, F=F, B=B, rel_margin=1e-4)
    knife = ref["fwd"]["knife"]
    dL = np.where(knife[..., None], 0, S.upstream_grad(r, cam.height, cam.width)).astype(np.float32)
    ref = O.step(cam, prm, sc, F=F, B=B, dL_dout=dL.astype(np.float64), rel_margin=1e-4)
    d = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to(dev())
    params = {k: d(v) for k, v in sc.items()}
    proj = api.project(cam, prm, **params)
    bins = api.bin_sort(cam.width, cam.height, proj)
    bins["tile_order"] = None
    split = api.make_split(bins["n_isect"] // 256 + api.n_tiles(*size) + 1, 256)
    fwd = api.render_fwd(cam, prm, bins, proj, F=d(F), B=d(B), split=split)
    grads = api.render_bwd(cam, prm, params, proj, bins, fwd, d(dL), F=d(F), B=d(B), split=split)
    torch.cuda.synchronize()
    assert np.abs(fwd["out"].cpu().numpy() - ref["fwd"]["out"])[~knife].max() <= 1e-5
    assert np.array_equal(fwd["last"].cpu().numpy().view(np.uint32)[~knife],
                          ref["fwd"]["last"][~knife])
    for k in params:
        g, gr = grads[k].cpu().numpy().astype(np.float64), ref["grads"][k]
        assert np.linalg.norm(g - gr) <= 1e-4 * max(np.linalg.norm(gr), 1e-30), k


@pytest.mark.parametrize("size", [(48, 48), (272, 256)])
def test_split_takes_slots_of_few_pairs(api, size):
    """A split forward takes a checkpoint slot for every chunk boundary that a walk
    crosses and one for the end of each tile split, however few pairs the lists
    hold in all; above 256 tiles its outputs are the unsplit ones bit by bit."""
    from paper_2608_27735_amd.camera import RasterParams, look_at
    r = S.rng(1100)
    cam = look_at((0.0, -3.0, 0.0), (0, 0, 0), *size)
    prm = RasterParams(sh_degree=0)
    sc = S.gaussians(r, r.uniform(-0.05, 0.05, (3000, 3)), 0, np.log(0.01), 0.3)
    sc["opacity_logits"] -= 5.0  # faint: the walks run through several chunks
    d = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to(dev())
    params = {k: d(v) for k, v in sc.items()}
    proj = api.project(cam, prm, **params)
    bins = api.bin_sort(cam.width, cam.height, proj)
    say("slots of few pairs", size, bins["n_isect"])
    assert bins["n_isect"] <= 65536
    split = api.make_split(bins["n_isect"] // 256 + api.n_tiles(*size) + 1, 256)
    fwd = api.render_fwd(cam, prm, bins, proj, split=split)
    whole = api.render_fwd(cam, prm, bins, proj)
    torch.cuda.synchronize()
    nty, ntx = (size[1] + 15) // 16, (size[0] + 15) // 16
    pad = np.zeros((16 * nty, 16 * ntx), np.int64)
    pad[:size[1], :size[0]] = fwd["last"].cpu().numpy()
    walk = pad.reshape(nty, 16, ntx, 16).max(axis=(1, 3))  # a lower bound: walks end past it
    crossed = np.maximum(walk - 1, 0) // 256
    assert crossed.max() >= 3
    taken = int(split["workspace"][:4].view(torch.int32))
    assert taken >= int(crossed.sum() + (crossed > 0).sum())
    if api.n_tiles(*size) > 256:
        for k in ("out", "final_T", "last"):
            assert torch.equal(fwd[k], whole[k])


@pytest.mark.parametrize("count", [127, 128, 129])
def test_backward_lists_about_the_rows_limit(api, count):
    """Lists one short of, at and one past the length from which the backward of an
    unsplit frame of 272 tiles gives a tile four workgroups instead of one."""
    test_forward_list_lengths(api, count, -4.0)


@pytest.mark.parametrize("bad", [np.nan, np.inf])
@pytest.mark.parametrize("at", ["middle", "edge"])
@pytest.mark.parametrize("size", [(203, 117), (270, 250), (523, 507)])
def test_backward_upstream_not_finite_stays_with_the_pixel(api, size, at, bad):
    """A NaN or an infinity in one pixel's upstream gradient reaches the Gaussians
    that this pixel blends and no other: not those that its wave or its group of
    four blends elsewhere, and, at the first pixel of a tile that the frame's edge
    cuts, nothing through the tile's pixels outside the frame. On 104 tiles (four
    workgroups a tile), 272 (one, without a schedule) and 1,056 (the queue)."""
    from paper_2608_27735_amd.camera import RasterParams, look_at
    r = S.rng(1200)
    cam = look_at((0.0, -3.0, 0.0), (0, 0, 0), *size)
    pos = np.stack([r.uniform(-1.8, 1.8, 4001), r.uniform(-0.5, 0.5, 4001), r.uniform(-1.8, 1.8, 4001)], 1)
    sc = S.gaussians(r, pos, 0, np.log(0.03), 0.5)
    prm = RasterParams(sh_degree=0)
    x, y = ((size[0] // 2, size[1] // 2) if at == "middle" else
            ((size[0] - 1) // 16 * 16, (size[1] - 1) // 16 * 16))
    say("not finite upstream", size, at, bad, x, y)
    d = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(dev())
    params = {k: d(v) for k, v in sc.items()}
    proj = api.project(cam, prm, **params)
    bins = api.bin_sort(cam.width, cam.height, proj)
    fwd = api.render_fwd(cam, prm, bins, proj)
    dL = S.upstream_grad(r, cam.height, cam.width)
    clean = api.render_bwd(cam, prm, params, proj, bins, fwd, d(dL))
    dL[y, x] = bad
    got = api.render_bwd(cam, prm, params, proj, bins, fwd, d(dL))
    torch.cuda.synchronize()
    # alphas of the pixel's walk in 64 bits
    ntx = (cam.width + 15) // 16
    a, _ = bins["tile_ranges"].cpu().numpy()[y // 16 * ntx + x // 16]
    walk = bins["values"].cpu().numpy()[a:a + int(fwd["last"][y, x])]
    u, v = proj["means2d"].cpu().numpy()[walk].astype(np.float64).T
    l11, l21, l22, o = proj["conic_opacity"].cpu().numpy()[walk].astype(np.float64).T
    dx, dy = x + 0.5 - u, y + 0.5 - v
    alpha = o * np.exp(-0.5 * ((l11 * dx + l21 * dy) ** 2 + (l22 * dy) ** 2))
    blended, near = np.zeros(4001, bool), np.zeros(4001, bool)
    blended[walk[alpha >= prm.alpha_min * (1 + 1e-4)]] = True
    near[walk[alpha >= prm.alpha_min * (1 - 1e-4)]] = True
    assert 0 < blended.sum() < len(walk)
    # the colour of a Gaussian that the pixel blends takes the pixel's gradient
    assert not torch.isfinite(got["sh"]).reshape(4001, -1).all(1).cpu().numpy()[blended].any()
    for k in params:
        g, c = got[k].cpu().numpy().reshape(4001, -1), clean[k].cpu().numpy().reshape(4001, -1)
        assert np.isfinite(g[~near]).all(), (k, int((~np.isfinite(g[~near]).all(1)).sum()))
        # the order of the atomic adds differs between the two calls
        assert np.linalg.norm(g[~near] - c[~near]) <= 1e-5 * np.linalg.norm(c), k


@pytest.mark.parametrize("size", [(128, 128), (272, 256), (528, 512)])
def test_opacity_below_the_normal_range(api, size):
    """Opacities that fp32 holds only as subnormal numbers, in the lists of an
    alpha_min below them, beside ordinary ones: finite gradients, at the parity
    bar of the oracle's, on each of the three backward kernels."""
    from paper_2608_27735_amd.camera import RasterParams, look_at
    r = S.rng(1300)
    cam = look_at((0.0, -3.0, 0.0), (0, 0, 0), *size)
    prm = RasterParams(sh_degree=0, alpha_min=1e-40)
    sc = S.gaussians(r, r.uniform(-0.8, 0.8, (601, 3)), 0, np.log(0.03), 0.3)
    sc["opacity_logits"][::2] = -88.0
    say("subnormal opacities", size)
    dL = S.upstream_grad(r, cam.height, cam.width)
    ref = O.step(cam, prm, sc, dL_dout=None, rel_margin=1e-4)
    dL = np.where(ref["fwd"]["knife"][..., None], 0, dL).astype(np.float32)
    ref = O.step(cam, prm, sc, dL_dout=dL.astype(np.float64), rel_margin=1e-4)
    d = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to(dev())
    params = {k: d(v) for k, v in sc.items()}
    proj = api.project(cam, prm, **params)
    o = proj["conic_opacity"][::2, 3]
    assert 0 < float(o.max()) < 2.0 ** -126
    assert int(proj["tiles_touched"][::2].sum()) > 0
    bins = api.bin_sort(cam.width, cam.height, proj)
    fwd = api.render_fwd(cam, prm, bins, proj)
    grads = api.render_bwd(cam, prm, params, proj, bins, fwd, d(dL))
    torch.cuda.synchronize()
    for k in params:
        g, gr = grads[k].cpu().numpy().astype(np.float64), ref["grads"][k]
        assert np.isfinite(g).all(), k
        assert np.linalg.norm(g - gr) <= 1e-4 * max(np.linalg.norm(gr), 1e-30), k


@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("count", [4, 5, 255, 257, 1023, 1024, 1029, 2051, 3072, 3075, 5121])
def test_adam_rows_of_the_last_workgroup(api, count, offset):
    """Counts that leave a group's last workgroup one to four rows of float4, whole
    and not, and up to three elements behind them."""
    test_adam_workgroup_edges(api, count, offset)


def test_binning_workgroup_memory_on_each_device(api):
    """The largest workgroup memory of each binning path on every device of the
    process, one after the other: the limit of dynamic memory is each device's own."""
    from paper_2608_27735_amd.camera import RasterParams, look_at
    for n, size in ((8192, (203, 117)), (9000, (203, 117)), (9000, (16, 16 * 32768))):
        r = S.rng(1400 + n)
        cam = look_at((0.2, -3.0, 0.9), (0, 0, 0), *size)
        sc = S.gaussians(r, r.uniform(-1.5, 1.5, (n, 3)), 0, np.log(0.02), 0.6)
        prm = RasterParams(sh_degree=0)
        pb = O.project_bin(cam, prm, sc["means"], sc["log_scales"], sc["quats"], sc["opacity_logits"])
        keys, values, ranges = O.bin(cam.width, cam.height, pb["depth"], pb["rect"], pb["tiles_touched"])
        for k in range(torch.cuda.device_count()):
            say("workgroup memory", k, n, size)
            with torch.cuda.device(k):
                proj = api.project(cam, prm, **{a: torch.from_numpy(v).to(f"cuda:{k}") for a, v in sc.items()})
                b = api.bin_sort(cam.width, cam.height, proj)
                torch.cuda.synchronize()
                assert np.array_equal(b["values"][:len(values)].cpu().numpy().view(np.uint32), values)
                assert np.array_equal(b["tile_ranges"].cpu().numpy().view(np.uint32), ranges)


@pytest.mark.parametrize("size", [(203, 117), (1280, 400)])
@pytest.mark.parametrize("n", [64, 255, 257, 513, 2047, 2048])
def test_binning_collect_of_one_round(api, n, size):
    """Blocks of up to 2,048 Gaussians, whose rectangles the collection holds in
    registers: quarters of one to eight rounds of 64 positions, whole and not."""
    test_binning_small_block_sizes(api, n, size)


@pytest.mark.parametrize("value", [1, 1 << 20])
@pytest.mark.parametrize("n", [700, 2048, 2049, 8192, 8193])
def test_binning_takes_tiles_touched_as_a_flag(api, n, value):
    """A tiles_touched that only tells the Gaussians with a tile from those without:
    the lists, and the count that the capacity is held against, are those of the
    boxes, on every path; nothing is written past the capacity."""
    from paper_2608_27735_amd.camera import RasterParams, look_at
    r = S.rng(1500 + n)
    cam = look_at((0.2, -3.0, 0.9), (0, 0, 0), 203, 117)
    sc = S.gaussians(r, r.uniform(-1.5, 1.5, (n, 3)), 0, np.log(0.03), 0.6)
    say("tiles as a flag", n, value)
    proj = api.project(cam, RasterParams(sh_degree=0),
                       **{k: torch.from_numpy(v).to(dev()) for k, v in sc.items()})
    want = api.bin_sort(cam.width, cam.height, proj)
    m = want["n_isect"]
    assert m == int(proj["tiles_touched"].sum())
    flag = dict(proj, tiles_touched=torch.where(proj["tiles_touched"] != 0, value, 0).to(torch.int32))
    for capacity in (m, m - 1):
        values = torch.full((m + 4096,), -7, dtype=torch.int32, device=dev())
        got = api.bin_sort(cam.width, cam.height, flag, capacity=capacity, values=values, sync=False)
        assert api.intersections(got["workspace"]) == m
        if capacity == m:
            assert torch.equal(got["tile_ranges"], want["tile_ranges"])
            assert torch.equal(values[:m], want["values"][:m])
            assert int((values[m:] != -7).sum()) == 0
        else:
            assert int(got["tile_ranges"].abs().max()) == 0 and int((values != -7).sum()) == 0


@pytest.mark.parametrize("size", [(151, 141), (275, 250), (530, 509)])
def test_walks_past_the_pixels_that_have_stopped(api, size):
    """An opaque cluster of small Gaussians before faint wide ones: the cluster's
    pixels stop within the first batches, those at its rim and beyond walk on, so
    each wave's box of pixels that still blend shrinks to a few columns and rows,
    to nothing, or stays whole. Split (151x141), and unsplit with the backward that
    takes tiles whole, directly and from the queue. Parity bars against the oracle."""
    from paper_2608_27735_amd.camera import RasterParams, look_at
    r = S.rng(1600)
    cam = look_at((0.0, -3.0, 0.0), (0, 0, 0), *size)
    prm = RasterParams(sh_degree=0)
    near = S.gaussians(r, np.stack([0.12 * r.standard_normal(2600), r.uniform(-0.6, -0.2, 2600),
                                    0.12 * r.standard_normal(2600)], 1), 0, np.log(0.012), 0.5)
    near["opacity_logits"] += 1.5
    far = S.gaussians(r, np.stack([r.uniform(-0.5, 0.5, 400), r.uniform(0.2, 0.6, 400),
                                   r.uniform(-0.5, 0.5, 400)], 1), 0, np.log(0.06), 0.5)
    far["opacity_logits"] -= 3.0
    sc = {k: np.concatenate([near[k], far[k]]) for k in near}
    F, B = S.background_pair(r, cam.height, cam.width)
    say("stopped pixels", size)
    ref = O.step(cam, prm, sc, F=F, B=B, rel_margin=1e-4)
    knife = ref["fwd"]["knife"]
    dL = np.where(knife[..., None], 0, S.upstream_grad(r, cam.height, cam.width)).astype(np.float32)
    ref = O.step(cam, prm, sc, F=F, B=B, dL_dout=dL.astype(np.float64), rel_margin=1e-4)
    last = ref["fwd"]["last"].astype(np.int64)
    pad = np.zeros((-(-cam.height // 8) * 8, -(-cam.width // 8) * 8), np.int64)
    pad[:cam.height, :cam.width] = last
    quad = pad.reshape(pad.shape[0] // 8, 8, pad.shape[1] // 8, 8).transpose(0, 2, 1, 3).reshape(-1, 64)
    # quadrants of which only some pixels walk past the end of a batch
    some = np.stack([(quad > b).sum(1) for b in range(256, int(quad.max()), 256)])
    assert ((some > 0) & (some < 32)).sum() >= 4 and (ref["fwd"]["final_T"][ref["fwd"]["last"] > 0] < 1e-3).any()
    d = lambda x: torch.from_numpy(np.ascontiguousarray(x)).to(dev())
    params = {k: d(v) for k, v in sc.items()}
    proj = api.project(cam, prm, **params)
    bins = api.bin_sort(cam.width, cam.height, proj)
    split = api.make_split(bins["n_isect"] // 256 + api.n_tiles(*size) + 1, 256) if size == (151, 141) else None
    fwd = api.render_fwd(cam, prm, bins, proj, F=d(F), B=d(B), split=split)
    grads = api.render_bwd(cam, prm, params, proj, bins, fwd, d(dL), F=d(F), B=d(B), split=split)
    torch.cuda.synchronize()
    assert np.abs(fwd["out"].cpu().numpy() - ref["fwd"]["out"])[~knife].max() <= 1e-5
    assert np.array_equal(fwd["last"].cpu().numpy().view(np.uint32)[~knife], ref["fwd"]["last"][~knife])
    for k in params:
        g, gr = grads[k].cpu().numpy().astype(np.float64), ref["grads"][k]
        assert np.linalg.norm(g - gr) <= 1e-4 * max(np.linalg.norm(gr), 1e-30), k
