"""GPU parity at the sizes where single kernels and dispatch branches can go
wrong: edges of tiles, remainders, the smallest and largest of a range."""
import numpy as np
import pytest
import torch

import oracle
import scenegen
from parity import assert_parity, compare

pytestmark = pytest.mark.gpu

DEV = torch.device("cuda:0")


def _native():
    from paper_2604_05794_amd import native
    native.lib()
    return native


def _t(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


@pytest.mark.parametrize("samples,patch,top_k", [(1, 1, 5), (5, 7, 5), (6, 5, 5), (16, 3, 8), (16, 7, 2)])
def test_paper_candidate_layers(samples, patch, top_k):
    """The five- and the sixteen-layer kernels, every patch size."""
    nat = _native()
    sc = scenegen.make_scene("tiny", 3)
    kw = dict(patch=patch, top_k=top_k)
    fp = dict(lam=3.0, n_samples=samples, delta=5e-3)
    pts = sc.points[:3997]
    d, c = nat.fuse_directions(_t(pts), _t(sc.cams), _t(sc.theta), _t(sc.conf), depth_maps=_t(sc.depth),
                               mode=nat.FD_MODE_FPMVO, fpmvo_lambda=fp["lam"], fpmvo_samples=samples,
                               fpmvo_delta=fp["delta"], **kw)
    torch.cuda.synchronize()
    orc = oracle.Oracle(sc.cams, sc.theta, sc.conf, depth=sc.depth, **kw)
    do, co = orc.fpmvo(pts, **fp)
    assert_parity(compare(orc, pts, d.cpu().numpy(), c.cpu().numpy(), do, co))


@pytest.mark.parametrize("dims,max_steps,bend,mode", [
    ((1, 1, 1), 1, -2.0, 0), ((2, 5, 3), 63, -2.0, 1), ((4, 4, 4), 64, 0.5, 2), ((9, 3, 130), 62, -2.0, 0),
    ((40, 40, 40), 127, -2.0, 1), ((40, 40, 40), 130, 0.9, 2), ((17, 16, 15), 65, 1.0, 0)])
def test_growing_bit_for_bit(dims, max_steps, bend, mode):
    """Traces identical to the oracle's on grids smaller and larger than the
    blocks that a wave loads, at lengths around the 64 vertices it stores at
    once, with seeds on voxel faces and outside the grid; bend 1.0: a voxel's
    orientation may fail the bend test against itself."""
    nat = _native()
    rng = np.random.default_rng(sum(dims) + max_steps)
    nx, ny, nz = dims
    d = rng.normal(size=(nz, ny, nx, 3)) * 0.35 + np.array([0.3, -0.5, 0.8])
    d /= np.linalg.norm(d, axis=-1, keepdims=True)
    d = (d * rng.choice([-1.0, 1.0], size=(nz, ny, nx, 1))).astype(np.float32)
    d[rng.uniform(size=(nz, ny, nx)) < 0.01] = 0.0
    occ = (rng.uniform(size=(nz, ny, nx)) > 0.02).astype(np.uint32)
    coh = rng.uniform(0.1, 1.0, size=(nz, ny, nx)).astype(np.float32)
    grid = (np.array([-0.013, 0.002, -0.3], np.float32), np.float32(0.0031), np.array(dims, np.int32))
    n = 301
    seeds = rng.uniform(-0.1, 1.1, size=(n, 3)) * np.array(dims) * 0.0031 + grid[0]
    seeds[:60] = np.round((seeds[:60] - grid[0]) / 0.0031) * np.float32(0.0031) + grid[0]
    seeds = seeds.astype(np.float32)
    sdirs = rng.normal(size=(n, 3)).astype(np.float32)
    cr = torch.from_numpy(rng.integers(0, 3, size=occ.size).astype(np.int32)).to(DEV)
    kw = dict(step=7e-4, max_steps=max_steps, min_coherence=0.12, max_bend_cos=bend, voxel_cap=9, batch=100)
    o = oracle.grow(dict(occ=occ, dir=d, coherence=coh), grid, seeds, sdirs if mode == 0 else None,
                    crossings=cr.cpu().numpy().view(np.uint32).copy(), seed_mode=mode, centre=(0.0, 0.0, 0.0), **kw)
    v, nv, last = nat.grow_strands(_t(occ.view(np.int32)), _t(d), _t(coh), *grid, _t(seeds), _t(sdirs) if mode == 0 else None,
                                   crossings=cr, seed_mode=mode, **kw)
    torch.cuda.synchronize()
    v, nv = v.cpu().numpy(), nv.cpu().numpy()
    assert np.array_equal(nv, o["n_verts"])
    for i in range(n):
        assert np.array_equal(v[i, :nv[i]], o["verts"][i, :nv[i]]), i
    assert np.array_equal(last.cpu().numpy(), o["last_dir"])
    assert np.array_equal(cr.cpu().numpy().view(np.uint32), o["crossings"])


@pytest.mark.parametrize("batch", [32, 96, 4096, 4128, 8224])
def test_training_batches(batch):
    """Gradients against the bfloat16 oracle (tolerances of the gradient
    test) at a padded row tile, the last batch of 16-row workgroups, the
    first of 32-row ones and a batch that cannot be split; then an Adam step,
    after which the matrix-core copies of the weights have to be the master
    weights'."""
    nat = _native()
    rng = np.random.default_rng(batch)
    parts = []
    for (W, b) in oracle.mlp_split(np.zeros(oracle.mlp_n_params())):
        parts += [rng.normal(0, 1.0 / np.sqrt(W.shape[0]), W.size), rng.normal(0, 0.1, b.size)]
    p = np.concatenate(parts).astype(np.float32)
    x = oracle.round_bf16(rng.normal(0, 1, (batch, 112)).astype(np.float32))
    t = rng.normal(size=(batch, 3))
    t = (t / np.linalg.norm(t, axis=1, keepdims=True)).astype(np.float32)
    net = nat.MLP(seed=0)
    net.set_params(p)
    xd = _t(x).to(torch.bfloat16)
    loss, grad = net.loss_grad(xd, _t(t))
    g = grad.cpu().numpy().astype(np.float64)
    lo, go = oracle.mlp_loss_grad(p.astype(np.float64), x, t, bf16=True)
    assert abs(float(loss.item()) - lo) <= 1e-3 * max(1.0, abs(lo))
    off = 0
    for (W, b) in oracle.mlp_split(np.zeros(oracle.mlp_n_params())):
        for size in (W.size, b.size):
            r = go[off:off + size]
            assert np.linalg.norm(g[off:off + size] - r) <= 1e-2 * np.linalg.norm(r), off
            off += size
    step_loss = torch.empty(1, device=DEV)
    net.train_step(xd, _t(t), lr=1e-3, loss=step_loss)
    assert float(step_loss.item()) == float(loss.item())
    other = nat.MLP(seed=1)
    other.set_params(net.get_params())
    assert torch.equal(net.forward(xd), other.forward(xd))
    a, b = net.loss_grad(xd, _t(t)), other.loss_grad(xd, _t(t))
    assert torch.equal(a[1], b[1]) and torch.equal(a[0], b[0])


@pytest.mark.parametrize("radius", range(1, 13))
def test_orientation_maps_radii_and_ranges(radius):
    """Every tap layout at sizes around the 16 x 64 tile, on frames of any
    scale: noise, a constant (responses are rounding), one pixel 2^40 times
    the others (below what the split halves hold), and non-finite pixels,
    which stay in their window.  Responses and confidences within the bounds
    of the orientation-map tests; the orientation is that of the binary32 sum
    over the taps in order, also where rounding decides."""
    import test_gpu_gabor as G
    rng = np.random.default_rng(radius)
    kw = dict(n_orient=(8, 16, 32)[radius % 3], radius=radius)
    h, w = 64 + radius % 3 - 1, 32 + (radius // 3) % 3 - 1
    base = rng.uniform(0.0, 1.0, (h, w))
    frames = np.stack([255.0 * base, 1e-3 * base, np.full((h, w), 0.7), base, base - 0.5]).astype(np.float32)
    frames[3] *= 2.0**-20
    frames[3, 40, 20] = 2.0**20
    frames[4, :, :8] *= 2.0**-30
    th, cf = G._gpu(frames, **kw)
    # the parameters as the entry point holds them
    bank = oracle.gabor_bank(**{k: v if k in kw else float(np.float32(v)) for k, v in G._bank_kw(kw).items()})
    for v in range(5):
        G._check_frame(frames[v], th[v], cf[v], bank, max_tie_frac=1.0)
        pad = np.pad(frames[v], radius).astype(np.longdouble)
        acc = np.zeros((kw["n_orient"], h, w), np.float32)
        for dy in range(2 * radius + 1):
            for dx in range(2 * radius + 1):
                tap = bank[:, dy, dx].astype(np.float32).astype(np.longdouble)
                acc = (tap[:, None, None] * pad[dy:dy + h, dx:dx + w] + acc).astype(np.float32)
        assert np.array_equal(np.rint(th[v] * kw["n_orient"] / np.pi), np.abs(acc).argmax(0))
    for bad in (np.nan, np.inf):
        f = frames[4].copy()
        f[30, 9] = bad
        tb, cb = G._gpu(f[None], **kw)
        inside = np.zeros((h, w), bool)
        inside[max(0, 30 - radius):31 + radius, max(0, 9 - radius):10 + radius] = True
        assert np.array_equal(tb[0][~inside], th[4][~inside])
        assert np.isnan(cb[0][inside]).all() and np.isfinite(cb[0][~inside]).all()


@pytest.mark.parametrize("dims,n", [((1, 1, 1), 1), ((1, 1, 1), 24), ((1, 1, 1), 25), ((1, 1, 1), 33), ((2, 1, 1), 48),
                                    ((2, 1, 1), 1003), ((3, 3, 3), 27 * 24), ((3, 3, 3), 27 * 40), ((64, 64, 1), 9000),
                                    ((17, 241, 1), 5000), ((16, 16, 16), 4096 * 30)])
def test_volume_slots_and_lanes(dims, n):
    """Around the 24 points a voxel at which a voxel gets eight lanes, counts
    that leave a remainder, one block of voxels more or less than whole.  The
    bounds of the volume tests."""
    import test_gpu_volume as V
    rng = np.random.default_rng(n)
    h = np.float32(0.01)
    pts = (rng.uniform(0.0, 1.0, (n, 3)) * np.array(dims) * 0.0099999).astype(np.float32)
    d = rng.normal(size=(n, 3)) + np.array([2.0, 0.5, -1.0])
    d = (d / np.linalg.norm(d, axis=1, keepdims=True)).astype(np.float32)
    w = rng.uniform(-0.1, 1.1, n).astype(np.float32)
    grid = (np.zeros(3, np.float32), h, np.array(dims, np.int32))
    o, *out, _, _ = V._compare(pts, d, *grid, np.clip(w, 0.0, 1.0))
    assert o["inside"] == n
    # weights outside [0, 1] act as the nearest (the oracle takes them as they are)
    for a, b in zip(out, V._gpu(pts, d, *grid, w)):
        assert np.array_equal(a, b)


@pytest.mark.parametrize("half", [False, True])
@pytest.mark.parametrize("views", [1, 15, 16, 17, 40, 128, 131])
def test_feature_rows_and_lists(views, half):
    """Fewer and more views than slots, some of them the same camera again
    (equal keys: the lower view first); point counts around those that a wave
    takes, on either side of the 65,536 from which it takes more.  Every count
    gives the rows that one call over all points gives, and those are the
    oracle's: the same slots, values within a bfloat16 step (of the 7504, four
    may miss it: the share that the feature test grants is 1e-4)."""
    nat = _native()
    rec = dict(scenegen.RECIPES["tiny"])
    rec.update(n_views=24, arc_deg=360.0)
    sc = scenegen.make_scene(rec, 5)
    v = np.arange(views) % 24
    v[2::3] = v[1::3][:len(v[2::3])]
    th, cf, dm = sc.theta[v], sc.conf[v], sc.depth[v]
    if half:
        th, cf, dm = (a.astype(np.float16) for a in (th, cf, dm))
    maps = (_t(sc.cams[v]), _t(th), _t(cf))
    kw = dict(head_centre=sc.head_centre, depth_maps=_t(dm))
    few = np.asarray(sc.points[:67], np.float32)
    pts = _t(np.resize(few, ((1 << 16) + 1 if views == 40 else 67, 3)))
    rows = nat.features(pts, *maps, **kw)
    head = rows[:67]
    if views == 40:  # the points repeat
        assert torch.equal(rows, head.repeat(len(pts) // 67 + 1, 1)[:len(pts)])
        assert torch.equal(nat.features(pts[:-1].contiguous(), *maps, **kw), rows[:-1])
    for n in (1, 3, 15, 16, 17, 63, 64, 65):
        assert torch.equal(nat.features(pts[:n].contiguous(), *maps, **kw), head[:n]), n
    f = head.float().cpu().numpy().astype(np.float64)
    fo = oracle.Oracle(sc.cams[v], th.astype(np.float32), cf.astype(np.float32), patch=1,
                       depth=dm.astype(np.float32)).features(few, sc.head_centre)
    assert np.array_equal(f[:, 6::7], fo[:, 6::7])
    err = np.abs(f - oracle.round_bf16(fo.astype(np.float32)).astype(np.float64))
    assert (err > 2.0 ** -7 * np.abs(fo) + 1e-5).sum() <= 4


@pytest.mark.parametrize("n", [1, 255, 257, 4095, 66000])
def test_setup_and_cell_ranks(n):
    """Point counts around a workgroup and above one round of the setup
    kernel (65,536 threads), points of one cell, a NaN: a point's result does
    not depend on the others, so every call gives the bits of its part of one
    call over all."""
    nat = _native()
    sc = scenegen.make_scene("tiny", 7)
    few = np.asarray(sc.points[:997], np.float32)
    pts = np.resize(few, (n, 3)).copy()
    pts[n // 2:] += np.float32(1e-6)  # twice the cells' points, not the same
    kw = dict(depth_maps=_t(sc.depth), patch=3, n_candidates=32, refine_iters=3, top_k=3)
    maps = (_t(sc.cams), _t(sc.theta), _t(sc.conf))
    one = nat.fuse_directions(_t(pts), *maps, **kw)
    torch.cuda.synchronize()
    part = max(1, n // 3)
    for rows in (np.arange(part), np.arange(n)[::-1].copy()):
        d, c = nat.fuse_directions(_t(pts[rows]), *maps, **kw)
        assert torch.equal(d, one[0][_t(rows)]) and torch.equal(c, one[1][_t(rows)])
    bad = np.vstack([pts[:part], np.full((1, 3), np.nan, np.float32)])
    d, c = nat.fuse_directions(_t(bad), *maps, **kw)
    assert torch.equal(d[:-1], one[0][:part]) and torch.equal(c[:-1], one[1][:part])
    assert not d[-1].any() and torch.isinf(c[-1])


@pytest.mark.parametrize("patch", [1, 3, 5, 7])
@pytest.mark.parametrize("scale", [10, -19, -22, -30, 29, 32])
def test_patch_normalisation_ranges(patch, scale):
    """Confidences times a power of two scale every sample's form exactly and
    leave every decision as it is, so the directions are the same bits whether
    the short or the general normalisation is taken (within 2^-44 < n2 and
    a form below 2^60, outside, or both in one map: confidences reach down
    from 1).  Costs are 1 - S / K of the scaled sums."""
    nat = _native()
    sc = scenegen.make_scene("tiny", 11)
    pts = _t(sc.points[:1500])
    kw = dict(depth_maps=_t(sc.depth), patch=patch, n_candidates=48, refine_iters=6, top_k=4)
    th = _t(sc.theta.astype(np.float32))
    cf = sc.conf.astype(np.float32)
    d0, c0 = nat.fuse_directions(pts, _t(sc.cams), th, _t(cf), **kw)
    d1, c1 = nat.fuse_directions(pts, _t(sc.cams), th, _t(cf * np.float32(2.0 ** scale)), **kw)
    assert torch.equal(d0, d1)
    s0, s1 = 1.0 - c0.double(), (1.0 - c1.double()) * 2.0 ** -scale
    ok = torch.isfinite(c0)
    assert torch.equal(ok, torch.isfinite(c1))
    # both costs are rounded to binary32
    tol = 2.0 ** -24 * (1.0 + c0.double().abs() + (1.0 + c1.double().abs()) * 2.0 ** -scale)
    assert ((s0 - s1).abs() <= tol)[ok].all()


@pytest.mark.parametrize("mode", ["plain", "fpmvo", "batched"])
def test_fallback_count_outlives_other_modes(mode):
    """The fallback counters are those of the last learned call on a context:
    calls in the other modes leave them as they are."""
    nat = _native()
    sc = scenegen.make_scene("tiny", 2)
    n = sc.n_points
    maps = (_t(sc.cams), _t(sc.theta), _t(sc.conf))
    kw = dict(depth_maps=_t(sc.depth), patch=3, n_candidates=32, refine_iters=3, top_k=3)
    ctx = nat.Context(max_points=2 * n, max_views=2 * len(sc.cams), max_scenes=2)
    learned = dict(mode=nat.FD_MODE_LEARNED, proposal=nat.FD_PROPOSAL_NAN, fallback_cost=float("inf"), ctx=ctx)
    nat.fuse_directions(_t(sc.points), *maps, **learned, **kw)
    split = ctx.fallback_split()
    assert ctx.fallback_count() == sum(split) == n
    if mode == "batched":
        import test_gpu_batched as B
        nat.fuse_batched([B._dev_scene(sc), B._dev_scene(sc)], ctx, **{k: v for k, v in kw.items() if k != "depth_maps"})
    else:
        other = dict(plain=nat.FD_MODE_PLAIN, fpmvo=nat.FD_MODE_FPMVO)[mode]
        nat.fuse_directions(_t(sc.points), *maps, mode=other, ctx=ctx, **kw)
    assert ctx.fallback_count() == n and ctx.fallback_split() == split


@pytest.mark.parametrize("bad", [np.nan, np.inf, -np.inf])
@pytest.mark.parametrize("radius,n_orient", [(1, 32), (3, 16), (7, 8), (8, 32), (11, 16), (12, 32)])
def test_non_finite_pixels_on_a_black_background(bad, radius, n_orient):
    """A non-finite pixel reaches the pixels whose window holds it and no
    other, also where everything around it is 0 (a window of zeros has no
    response and no confidence)."""
    import test_gpu_gabor as G
    h, w = 150, 64
    img = np.zeros((h, w), np.float32)
    img[4:7, 5] = 1.0
    kw = dict(n_orient=n_orient, radius=radius)
    t0, c0 = G._gpu(img[None], **kw)
    for y, x in ((70, 30), (63, 16), (64, 47), (140, 60)):
        f = img.copy()
        f[y, x] = bad
        t1, c1 = G._gpu(f[None], **kw)
        inside = np.zeros((h, w), bool)
        inside[max(0, y - radius):y + radius + 1, max(0, x - radius):x + radius + 1] = True
        assert np.isnan(c1[0][inside]).all()
        assert np.array_equal(t1[0][~inside], t0[0][~inside])
        # a rescaled tile may take the same response from the other sum
        assert np.allclose(c1[0][~inside], c0[0][~inside], rtol=0.0, atol=2e-5)
        assert not c1[0][~inside][c0[0][~inside] == 0.0].any()


def _gabor_kinds(rng, h, w):
    """Frames that take every way through the orientation kernels: noise, low
    contrast (centred tiles; some of them in the binary32 kernel), a ramp and a
    constant (binary32), black with noise, halves of two kinds side by side, one
    pixel 2^40 times the others, 8 bits, negative values."""
    noise = rng.uniform(0.0, 1.0, (h, w))
    yy, xx = np.mgrid[0:h, 0:w]
    ramp = (xx + 0.3 * yy) / (w + h)
    lowc = 0.15 + 0.02 * rng.normal(size=(h, w))
    f = dict(noise=255.0 * noise, lowc=lowc, flat=0.8 + 0.002 * rng.normal(size=(h, w)), ramp=ramp,
             constant=np.full((h, w), 0.7), black=0.02 * rng.normal(size=(h, w)),
             sides=np.where(xx < w // 2 + 5, ramp, np.where(yy < h // 3, noise, lowc)), tiny=2.0**-20 * noise,
             bits8=np.round(255 * np.clip(0.5 + 0.3 * np.sin(0.9 * xx + 0.2 * yy) + 0.02 * rng.normal(size=(h, w)), 0, 1)) / 255,
             negative=-0.4 - 0.1 * noise)
    f["tiny"][h // 2, w // 2] = 2.0**20
    return {k: v.astype(np.float32) for k, v in f.items()}


@pytest.mark.parametrize("radius,n_orient", [(5, 32), (5, 16), (6, 8), (7, 16), (8, 32), (8, 16), (9, 32), (10, 8), (11, 32), (12, 32), (12, 16)])
def test_large_frames_choose_as_small_ones(radius, n_orient):
    """Frames of more than 640 tiles take the split sums (from radius 5 on), cut
    up they do not: the orientations are those of the binary32 sum in order,
    which the small frames' test pins, bit for bit wherever the window lies in
    the piece or the frame ends with it, and the confidences those of the
    oracle within its tests' bounds.  1.9 million pixels a kind, many times what
    the persistent workgroups hold at once."""
    import test_gpu_gabor as G
    nat = _native()
    rng = np.random.default_rng(100 * radius + n_orient)
    h, w = 1237, 1541  # 20 x 97 tiles, neither edge on a tile's
    kw = dict(n_orient=n_orient, radius=radius, out_dtype=torch.float32)
    kinds = _gabor_kinds(rng, h, w)
    frames = _t(np.stack(list(kinds.values())))
    theta, conf = nat.orientation_maps(frames, **kw)
    ph, pw = 252, 236  # 4 x 15 tiles
    wrong = {}
    for y0 in range(0, h, ph - 2 * radius):
        for x0 in range(0, w, pw - 2 * radius):
            y1, x1 = min(h, y0 + ph), min(w, x0 + pw)
            ya, yb = y0 + (radius if y0 else 0), y1 - (radius if y1 < h else 0)
            xa, xb = x0 + (radius if x0 else 0), x1 - (radius if x1 < w else 0)
            if ya >= yb or xa >= xb:
                continue
            t, _ = nat.orientation_maps(frames[:, y0:y1, x0:x1].contiguous(), **kw)
            off = (t[:, ya - y0:yb - y0, xa - x0:xb - x0] != theta[:, ya:yb, xa:xb]).flatten(1).sum(1)
            for name, c in zip(kinds, off.tolist()):
                wrong[name] = wrong.get(name, 0) + c
    assert not any(wrong.values()), wrong
    # one by one, the same bits
    for k in (0, 1, 6):
        t, c = nat.orientation_maps(frames[k:k + 1], **kw)
        assert torch.equal(t[0], theta[k]) and torch.equal(c[0], conf[k])
    # confidences against the oracle over a corner, where the frame's largest is put (bright noise)
    bank = oracle.gabor_bank(**{k: v if k in kw else float(np.float32(v)) for k, v in G._bank_kw(dict(n_orient=n_orient, radius=radius)).items()})
    n = 150
    for name in ("lowc", "flat", "sides", "black"):
        img = kinds[name].copy()
        img[:40, :60] = rng.uniform(0.0, 2.0, (40, 60)).astype(np.float32)
        t, c = nat.orientation_maps(_t(img[None]), **kw)
        part = img[:n + radius, :n + radius]
        t, c = t[0, :n, :n].cpu().numpy(), c[0, :n, :n].cpu().numpy()
        to, co, wmax, F = oracle.gabor(part, bank, responses=True)
        _, _, _, L1 = oracle.gabor(np.abs(part), np.abs(bank), responses=True)
        scale = L1.max(axis=-1)[:n, :n]
        co = co[:n, :n]
        jo, jt = (np.rint(v * n_orient / np.pi).astype(int)[..., None] for v in (to[:n, :n], t))
        same = (jo == jt)[..., 0]
        near = np.take_along_axis(F[:n, :n], jo, -1) - np.take_along_axis(F[:n, :n], jt, -1)
        assert (near[..., 0] <= 2 * G.REL * scale).all(), name
        k = np.arange(n_orient)
        dk = np.minimum(k, n_orient - k) * (np.pi / n_orient)
        dw = 2 * G.REL * scale * np.sqrt(np.sum(dk * dk))
        bound = dw / wmax + co * (dw.max() / wmax) + 1e-7
        assert (np.abs(c - co) <= bound)[same].all(), name


@pytest.mark.parametrize("n_orient,tiles", [(32, (16, 20)), (32, (16, 19)), (16, (16, 40)), (16, (16, 39)), (8, (1, 640)), (32, (320, 1))])
def test_orientation_frames_at_the_split_size(n_orient, tiles):
    """Frames of just the tiles from which the split sums are taken, and one
    row of tiles less; a single row and a single column of tiles: orientations
    of the pieces, and the same maps for a frame alone and among others."""
    nat = _native()
    rng = np.random.default_rng(n_orient + tiles[0])
    h, w = 64 * tiles[0] - 3, 16 * tiles[1] - 1
    f = _t(rng.uniform(0.0, 1.0, (3, h, w)).astype(np.float32))
    kw = dict(n_orient=n_orient, radius=8, out_dtype=torch.float32)
    theta, conf = nat.orientation_maps(f, **kw)
    t1, c1 = nat.orientation_maps(f[1:2].contiguous(), **kw)
    assert torch.equal(t1[0], theta[1]) and torch.equal(c1[0], conf[1])
    for y0 in range(0, h, 100):
        for x0 in range(0, w, 1000):
            y1, x1 = min(h, y0 + 116), min(w, x0 + 1016)
            t, _ = nat.orientation_maps(f[:, y0:y1, x0:x1].contiguous(), **kw)
            ya, yb = y0 + (8 if y0 else 0), y1 - (8 if y1 < h else 0)
            xa, xb = x0 + (8 if x0 else 0), x1 - (8 if x1 < w else 0)
            assert torch.equal(t[:, ya - y0:yb - y0, xa - x0:xb - x0], theta[:, ya:yb, xa:xb])


@pytest.mark.parametrize("bad", [np.nan, np.inf, -np.inf])
@pytest.mark.parametrize("radius,n_orient", [(5, 16), (8, 32), (11, 8), (12, 32)])
def test_non_finite_pixels_in_large_frames(bad, radius, n_orient):
    """As on a black background above, in frames that take the split sums: over
    black, over noise and over low contrast."""
    nat = _native()
    rng = np.random.default_rng(radius)
    h, w = 1030, 1100
    kw = dict(n_orient=n_orient, radius=radius, out_dtype=torch.float32)
    base = np.zeros((3, h, w), np.float32)
    base[0, 4:60, 5:40] = 1.0
    base[1] = rng.uniform(0.0, 1.0, (h, w))
    base[2] = 0.15 + 0.02 * rng.normal(size=(h, w))
    t0, c0 = nat.orientation_maps(_t(base), **kw)
    f = base.copy()
    inside = torch.zeros((h, w), dtype=torch.bool, device=DEV)
    for y, x in ((70, 30), (511, 512), (640, 655), (1020, 1099), (300, 0)):
        f[:, y, x] = bad
        inside[max(0, y - radius):y + radius + 1, max(0, x - radius):x + radius + 1] = True
    t1, c1 = nat.orientation_maps(_t(f), **kw)
    assert torch.isnan(c1[:, inside]).all() and torch.isfinite(c1[:, ~inside]).all()
    assert torch.equal(t1[:, ~inside], t0[:, ~inside])
    black = ~inside & (c0[0] == 0.0)
    assert not c1[0][black].any()


@pytest.mark.parametrize("samples", [6, 8, 9, 13, 16])
@pytest.mark.parametrize("patch,top_k", [(1, 5), (3, 5), (3, 2), (5, 5), (7, 8)])
def test_paper_candidate_rounds(samples, patch, top_k):
    """Layers held eight at a time, in one round and two, and all at once.  Points
    of at least two views: the candidates of a single one lie in its own plane,
    so that all layers tie; of those only the cost is compared."""
    nat = _native()
    sc = scenegen.make_scene("tiny", 4)
    kw = dict(patch=patch, top_k=top_k)
    fp = dict(lam=2.0, n_samples=samples, delta=8e-3)
    pts = sc.points[:2003]
    d, c = nat.fuse_directions(_t(pts), _t(sc.cams), _t(sc.theta), _t(sc.conf), depth_maps=_t(sc.depth),
                               mode=nat.FD_MODE_FPMVO, fpmvo_lambda=fp["lam"], fpmvo_samples=samples,
                               fpmvo_delta=fp["delta"], **kw)
    torch.cuda.synchronize()
    orc = oracle.Oracle(sc.cams, sc.theta, sc.conf, depth=sc.depth, **kw)
    do, co = orc.fpmvo(pts, **fp)
    d, c = d.cpu().numpy(), c.cpu().numpy()
    two = np.array([len(orc.select_views(p)[0]) > 1 for p in pts])
    assert_parity(compare(orc, pts[two], d[two], c[two], do[two], co[two]))
    assert np.allclose(c[~two], co[~two], rtol=0.0, atol=1e-5)


@pytest.mark.parametrize("part", ["every mantissa", "products", "outside"])
def test_sample_normalisation_is_rounded_as_ieee(part):
    """p / sqrt(n2) and q / sqrt(n2) against binary32 square root and division:
    every mantissa of n2 in two binades; the operands as a sample forms them, of
    confidences from 2^-22 to 2^30; and outside the short form's range, special
    values among them.  The same bits, apart from p and q below 2^-103 (an
    ulp)."""
    nat = _native()
    rng = np.random.default_rng(len(part))
    f = np.float32
    n = 1 << 24
    if part == "every mantissa":
        n2 = np.arange(n, dtype=np.uint32) + f(1.0).view(np.uint32)
        n2 = n2.view(f) * (f(2.0) ** (2 * rng.integers(-21, 30, n))).astype(f)
        al = np.full(n, 1.0, f)
        p = (rng.uniform(1.0, 2.0, n) * 2.0 ** rng.integers(-103, 92, n)).astype(f)
        q = -(rng.uniform(1.0, 2.0, n) * 2.0 ** rng.integers(-103, 92, n)).astype(f)
    elif part == "products":
        n = 1 << 22
        cb = (rng.uniform(1.0, 2.0, n) * 2.0 ** rng.integers(-23, 30, n)).astype(f)
        m = cb * rng.uniform(0.0, 1.0, n).astype(f) ** f(2.0)
        t = np.where(rng.uniform(size=n) < 0.2, rng.choice([0.0, 0.5, 1.0, 1.5], n) * np.pi + 10.0 ** rng.uniform(-40, -6, n),
                     rng.uniform(0, 2 * np.pi, n))
        mx, my = (m * np.cos(t)).astype(f), (m * np.sin(t)).astype(f)
        with np.errstate(all="ignore"):
            n2, al = mx * mx + my * my, f(0.5) * cb * cb
            p, q = al * mx, f(2.0) * al * my
    else:
        n = 1 << 20
        special = np.array([0.0, 1e-45, 2.0**-149, 2.0**-126, 2.0**-60, 2.0**-44, 1.0, 2.0**60, 2.0**61, 3e38, np.inf, np.nan], f)
        n2, al, p, q = (np.where(rng.uniform(size=n) < 0.5, rng.choice(special, n),
                                 (rng.uniform(1.0, 2.0, n) * 2.0 ** rng.integers(-120, 120, n)).astype(f)).astype(f) for _ in range(4))
        n2 = np.where((n2 > 2.0**-44) & (al < 2.0**60), f(2.0**-50) * np.minimum(n2, f(16.0)), n2).astype(f)
        q = -q
    got = [v.cpu().numpy() for v in nat.probe_norm(*map(_t, (n2, al, p, q)))]
    on = n2 > 0.0
    with np.errstate(all="ignore"):
        for g, x in zip(got, (p, q)):
            want = x / np.sqrt(n2)
            same = (g == want) | (np.isnan(g) & np.isnan(want))
            small = (np.abs(x) < 2.0**-103) & (n2 > 2.0**-44) & (al < 2.0**60)
            assert same[on & ~small].all(), int((~same & on & ~small).sum())
            assert (np.abs(g - want) <= np.spacing(np.abs(want)))[on & small].all()


@pytest.mark.parametrize("half", [False, True])
@pytest.mark.parametrize("views", [9, 64, 131])
def test_feature_rows_of_many_points(views, half):
    """Rows of 3001 distinct points against the oracle: the same slots, and the
    share of values off by more than a bfloat16 step that the feature test
    grants (1e-4), of 336,112."""
    nat = _native()
    rec = dict(scenegen.RECIPES["tiny"], n_points=3001, n_views=min(views, 48), arc_deg=360.0)
    sc = scenegen.make_scene(rec, 8)
    v = np.arange(views) % len(sc.cams)
    cams = sc.cams[v].copy()
    cams[len(sc.cams):, 13] += np.float32(1e-3)  # further views: a millimetre aside
    th, cf, dm = sc.theta[v], sc.conf[v], sc.depth[v]
    if half:
        th, cf, dm = (a.astype(np.float16) for a in (th, cf, dm))
    pts = np.asarray(sc.points, np.float32)
    rows = nat.features(_t(pts), _t(cams), _t(th), _t(cf), head_centre=sc.head_centre, depth_maps=_t(dm))
    f = rows.float().cpu().numpy().astype(np.float64)
    fo = oracle.Oracle(cams, th.astype(np.float32), cf.astype(np.float32), patch=1,
                       depth=dm.astype(np.float32)).features(pts, sc.head_centre)
    assert np.array_equal(f[:, 6::7], fo[:, 6::7])
    err = np.abs(f - oracle.round_bf16(fo.astype(np.float32)).astype(np.float64))
    assert (err > 2.0 ** -7 * np.abs(fo) + 1e-5).sum() <= 1e-4 * err.size


@pytest.mark.parametrize("mode,cap,bend", [(0, 0, -2.0), (1, 6, 0.5), (2, 3, 0.9)])
def test_growing_on_both_sides_of_the_lane_batch(mode, cap, bend):
    """8192 seeds take a wave each, 8193 two launches: the same traces as the
    oracle's, and as each other's over the seeds that both have."""
    nat = _native()
    rng = np.random.default_rng(mode)
    dims = (44, 37, 41)
    nx, ny, nz = dims
    d = rng.normal(size=(nz, ny, nx, 3)) * 0.3 + np.array([0.5, 0.2, -0.7])
    d /= np.linalg.norm(d, axis=-1, keepdims=True)
    d = (d * rng.choice([-1.0, 1.0], size=(nz, ny, nx, 1))).astype(np.float32)
    d[rng.uniform(size=(nz, ny, nx)) < 0.01] = 0.0
    d[5:8, :, :] *= np.float32(1e-25)  # an agreement that underflows
    occ = (rng.uniform(size=(nz, ny, nx)) > 0.02).astype(np.uint32)
    coh = rng.uniform(0.1, 1.0, size=(nz, ny, nx)).astype(np.float32)
    grid = (np.array([0.1, -0.07, 0.02], np.float32), np.float32(0.0027), np.array(dims, np.int32))
    n = 8193
    seeds = (rng.uniform(-0.02, 1.02, size=(n, 3)) * np.array(dims) * 0.0027 + grid[0]).astype(np.float32)
    sdirs = rng.normal(size=(n, 3)).astype(np.float32) if mode == 0 else None
    kw = dict(step=6e-4, max_steps=80, min_coherence=0.12, max_bend_cos=bend, voxel_cap=cap)
    got = []
    for batch in (8192, 8193):
        cr = torch.zeros(occ.size, dtype=torch.int32, device=DEV)
        v, nv, last = nat.grow_strands(_t(occ.view(np.int32)), _t(d), _t(coh), *grid, _t(seeds), None if sdirs is None else _t(sdirs),
                                       crossings=cr, seed_mode=mode, centre=(0.15, 0.0, 0.05), batch=batch, **kw)
        o = oracle.grow(dict(occ=occ, dir=d, coherence=coh), grid, seeds, sdirs, crossings=np.zeros(occ.size, np.uint32),
                        seed_mode=mode, centre=(0.15, 0.0, 0.05), batch=batch, **kw)
        v, nv, last = v.cpu().numpy(), nv.cpu().numpy(), last.cpu().numpy()
        on = np.arange(v.shape[1])[None] < nv[:, None]
        assert np.array_equal(nv, o["n_verts"]) and np.array_equal(last, o["last_dir"])
        assert np.array_equal(v[on], o["verts"][:, :v.shape[1]][on])
        assert np.array_equal(cr.cpu().numpy().view(np.uint32), o["crossings"])
        got.append((nv, v, on, last))
    (na, va, ona, la), (nb, vb, onb, lb) = got
    assert np.array_equal(na[:8192], nb[:8192]) and np.array_equal(la[:8192], lb[:8192])
    assert np.array_equal(va[:8192][ona[:8192]], vb[:8192][onb[:8192]])


@pytest.mark.parametrize("counts,singles", [([127, 128, 129, 300, 4001], 3000), ([5000], 1000), ([129] * 70, 600),
                                            ([1023, 1024, 1025, 6001, 31], 0), ([1025] * 20 + [1] * 5, 0)])
def test_volume_heavy_voxels(counts, singles):
    """Voxels around the points from which the whole wave takes one, few and
    many to a wave, with one lane a voxel (many single points) and eight.  The
    bounds of the volume tests."""
    import test_gpu_volume as V
    rng = np.random.default_rng(len(counts) + singles)
    dims = np.array([40, 30, 20])
    h = np.float32(0.01)
    at = rng.choice(int(np.prod(dims)), len(counts) + singles, replace=False)
    at = np.repeat(at, np.array(counts + [1] * singles))
    cell = np.stack([at % 40, at // 40 % 30, at // 1200], 1)
    pts = ((cell + rng.uniform(0.01, 0.99, cell.shape)) * 0.01).astype(np.float32)
    keep = rng.permutation(len(pts))
    d = rng.normal(size=(len(pts), 3)) + np.array([1.0, -0.4, 0.8])
    d = (d / np.linalg.norm(d, axis=1, keepdims=True)).astype(np.float32)
    w = rng.uniform(0.0, 1.0, len(pts)).astype(np.float32)
    V._compare(pts[keep], d[keep], np.zeros(3, np.float32), h, dims.astype(np.int32), w[keep])


@pytest.mark.parametrize("repeat", [2, 3, 64])
@pytest.mark.parametrize("views", [40, 64, 150])
def test_feature_lists_of_coinciding_cameras(views, repeat):
    """Cameras at the same place (with other orientations or the same, more of
    them than slots, mixed with cameras a rounding apart) leave the list in the
    order of the oracle's: by frontality, then by view."""
    nat = _native()
    rec = dict(scenegen.RECIPES["tiny"], n_points=500, n_views=24, arc_deg=360.0)
    sc = scenegen.make_scene(rec, 12)
    rng = np.random.default_rng(views + repeat)
    v = rng.permutation(np.arange(views) // repeat % 24)
    cams = sc.cams[v].copy()
    near = rng.uniform(size=views) < 0.3  # the last bit of the translation
    cams[near, 13] = np.nextafter(cams[near, 13], np.float32(np.inf))
    pts = np.asarray(sc.points, np.float32)
    rows = nat.features(_t(pts), _t(cams), _t(sc.theta[v]), _t(sc.conf[v]), head_centre=sc.head_centre)
    f = rows.float().cpu().numpy().astype(np.float64)
    fo = oracle.Oracle(cams, sc.theta[v].astype(np.float32), sc.conf[v].astype(np.float32), patch=1).features(pts, sc.head_centre)
    assert np.array_equal(f[:, 6::7], fo[:, 6::7])
    err = np.abs(f - oracle.round_bf16(fo.astype(np.float32)).astype(np.float64))
    assert (err > 2.0 ** -7 * np.abs(fo) + 1e-5).sum() <= 1e-4 * err.size


@pytest.mark.parametrize("n,far,max_steps", [(8193, 0.1, 33), (20011, 0.05, 70), (20011, 1.0, 32), (20011, 1.0, 33),
                                             (20011, 1.0, 100), (70001, 0.1, 65), (600_000, 0.005, 40)])
@pytest.mark.parametrize("mode", [0, 2])
def test_growing_large_batches(n, far, max_steps, mode):
    """One batch of more than 8192 seeds, few or most of which go further than
    the first steps, steps that end with them, one after them and past a
    block of 64 vertices: bit for bit the oracle's traces and crossings."""
    nat = _native()
    rng = np.random.default_rng(n + max_steps + mode)
    dims = (40, 36, 52)
    nx, ny, nz = dims
    z = np.arange(nz, dtype=np.float64)[:, None, None, None]
    d = np.concatenate([np.sin(z / 9), np.cos(z / 7), 1.5 + 0 * z], -1) + 0.15 * rng.normal(size=(nz, ny, nx, 3))
    d /= np.linalg.norm(d, axis=-1, keepdims=True)
    d = (d * rng.choice([-1.0, 1.0], size=(nz, ny, nx, 1))).astype(np.float32)
    occ = np.ones((nz, ny, nx), np.uint32)
    coh = np.ones((nz, ny, nx), np.float32)
    h = np.float32(0.003)
    grid = (np.array([-0.06, -0.05, -0.08], np.float32), h, np.array(dims, np.int32))
    seeds = (rng.uniform(0.05, 0.95, size=(n, 3)) * np.array(dims) * 0.003 + grid[0]).astype(np.float32)
    seeds[rng.uniform(size=n) >= far] += np.float32(1.0)  # outside
    sdirs = rng.normal(size=(n, 3)).astype(np.float32) if mode == 0 else None
    kw = dict(seed_mode=mode, centre=(0.01, 0.0, -0.02), step=1e-3, max_steps=max_steps, min_coherence=0.5,
              max_bend_cos=0.3, voxel_cap=4, batch=n)
    busy = np.where(rng.uniform(size=occ.size) < 0.001, 4, 0).astype(np.uint32)  # at the cap
    cr = _t(busy.view(np.int32).copy())
    v, nv, last = nat.grow_strands(_t(occ.view(np.int32)), _t(d), _t(coh), *grid, _t(seeds), None if sdirs is None else _t(sdirs),
                                   crossings=cr, **kw)
    o = oracle.grow(dict(occ=occ, dir=d, coherence=coh), grid, seeds, sdirs, crossings=busy.copy(), **kw)
    v, nv, last = v.cpu().numpy(), nv.cpu().numpy(), last.cpu().numpy()
    assert (o["n_verts"] > 33).mean() > 0.2 * far or max_steps <= 33
    assert np.array_equal(nv, o["n_verts"]) and np.array_equal(last, o["last_dir"])
    on = np.arange(v.shape[1])[None] < nv[:, None]
    assert np.array_equal(v[on], o["verts"][:, :v.shape[1]][on])
    assert np.array_equal(cr.cpu().numpy().view(np.uint32), o["crossings"])


@pytest.mark.parametrize("n_orient,radius", [(32, 8), (16, 3), (8, 12)])
@pytest.mark.parametrize("h", [1, 31, 32, 33, 64, 65, 81, 97, 129])
def test_orientation_rows_of_half_tiles(h, n_orient, radius):
    """Heights around the 32 rows of a half tile, in several small frames: each
    frame within the bounds of the orientation-map tests."""
    import test_gpu_gabor as G
    rng = np.random.default_rng(h)
    kw = dict(n_orient=n_orient, radius=radius)
    frames = rng.uniform(0.0, 1.0, (4, h, 53)).astype(np.float32)
    th, cf = G._gpu(frames, **kw)
    bank = oracle.gabor_bank(**{k: v if k in kw else float(np.float32(v)) for k, v in G._bank_kw(kw).items()})
    for v in range(4):
        G._check_frame(frames[v], th[v], cf[v], bank, max_tie_frac=1.0)
