"""The work that a user of the library has it do, as cases that can be timed and compared.

listed() and draw() give cases, prepare() what a program holds before the call, run() one pass through
the public entry points, work() what a pass cannot do without, exact() the same outputs in 64 bits.
"""
import math
import struct

import numpy as np
import torch

from paper_2604_05794_amd import native

DEV = "cuda:0"
WEIGHTS = "paper_2604_05794_amd/weights/proposal_mlp.fdmlp"
SCALP = 0.10  # radius of the head (m)
VIS_TAU = 5e-3  # visibility tolerance (m)
GROW = dict(step=1e-3, max_steps=200, min_coherence=0.1, max_bend_cos=math.cos(math.radians(45.0)), voxel_cap=8)
LINK = dict(max_dist=3e-3, min_cos=math.cos(math.radians(30.0)))
SEARCH = dict(hair="mixed", noise=0.14, outliers=0.1, depth=True, arc=360, patch=5, candidates=128, iters=8, top_k=5)
CURLS = dict(SEARCH, hair="curls", noise=0.32, outliers=0.3)


def listed():
    return [
        # a first look at a capture: few views of a small scene, where launches count
        dict(SEARCH, name="small_scene_f32", kind="search", mode="plain", points=10_000, views=12, res=256, strands=200, half=False,
             hair="helix", noise=0.14, outliers=0.0, arc=120, patch=3, candidates=48),
        # one captured hairstyle at full resolution: the plain search
        dict(SEARCH, name="scene_f16", kind="search", mode="plain", points=500_000, views=64, res=1024, strands=20_000, half=True),
        # the same kind of capture through the paper's own candidates (offset pixel, depth layers, medoid)
        dict(SEARCH, name="paper_candidates_f16", kind="search", mode="fpmvo", points=150_001, views=64, res=1024, strands=10_000, half=True),
        # one head of tight curls through the learned form
        dict(CURLS, name="head_learned_f16", kind="search", mode="learned", points=250_000, views=128, res=1024, strands=8_000, half=True),
        # eight such heads in one launch, the shape that tuning picks for them: the headline workload
        dict(CURLS, name="heads_batched_learned", kind="batch", mode="learned", scenes=8, points=2_000_000, ratio=1.0, views=128,
             res=1024, strands=8_000, half=True, tuned=True),
        # a batch of uneven hairstyles, plain search, shape not tuned
        dict(SEARCH, name="hairstyles_batched_plain", kind="batch", mode="plain", scenes=8, points=1_000_000, ratio=16.0, views=96,
             res=1024, strands=6_000, half=True, tuned=False),
        # network inputs of a float32 capture without depth maps, as the training data is made
        dict(name="features_f32", kind="features", points=60_001, views=96, res=768, strands=4_000, half=False, hair="mixed", noise=0.14,
             outliers=0.1, depth=False, arc=360),
        # the proposal network by itself over the points of four hairstyles
        dict(name="proposals", kind="forward", rows=1_000_003),
        # training between two looks at the weights: 16 Adam steps
        dict(name="training", kind="train", batch=4096, steps=16),
        # the orientation and confidence maps of a 64-frame capture
        dict(name="maps_64_frames", kind="maps", frames=64, width=1024, height=1024, orient=32, radius=8, half=True),
        # the volume of a hairstyle's outer and inner points at the paper's finest voxel
        dict(name="volume_2mm", kind="volume", points=2_000_000, voxel=0.002, weights=True, tensor=False),
        # a whole head of hair grown through a volume, linked and put together
        dict(name="strands_20k", kind="strands", points=8_000_000, voxel=0.003, roots=20_000, stride=3, batch=4096),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["search", "search", "search", "batch", "features", "forward", "train", "maps", "volume", "strands"])
    if kind == "search":
        mode = rng.choice(["plain", "plain", "learned", "fpmvo"])
        patch, k, cand, iters = rng.choice([1, 3, 5, 5, 7]), rng.choice([1, 3, 5, 5, 5, 8]), _log(rng, 16, 300), rng.randint(3, 10)
        per = (cand + 6 * iters) * k * patch * patch
        return dict(kind=kind, mode=mode, points=_log(rng, 500, min(500_000, int(2e10 / per))), views=rng.randint(8, 140), res=_log(rng, 160, 1024),
                    strands=_log(rng, 200, 15_000), half=rng.random() < 0.7, hair=rng.choice(["mixed", "curls", "helix"]),
                    noise=rng.uniform(0.05, 0.35), outliers=rng.uniform(0.0, 0.3), depth=mode == "fpmvo" or rng.random() < 0.8,
                    arc=rng.choice([120, 360]), patch=patch, candidates=cand, iters=iters, top_k=k)
    if kind == "batch":
        base = dict(rng.choice([SEARCH, CURLS]))
        return dict(base, kind=kind, mode=rng.choice(["plain", "learned"]), scenes=rng.randint(2, 10), points=_log(rng, 5_000, 1_000_000),
                    ratio=rng.choice([1.0, 4.0, 16.0]), views=rng.randint(12, 128), res=_log(rng, 256, 1024), strands=_log(rng, 500, 6_000),
                    half=rng.random() < 0.8, tuned=rng.random() < 0.5)
    if kind == "features":
        return dict(kind=kind, points=_log(rng, 500, 300_000), views=rng.randint(8, 160), res=_log(rng, 160, 1024), strands=_log(rng, 300, 8_000),
                    half=rng.random() < 0.6, hair=rng.choice(["mixed", "curls"]), noise=rng.uniform(0.05, 0.35), outliers=rng.uniform(0.0, 0.3),
                    depth=rng.random() < 0.6, arc=360)
    if kind == "forward":
        return dict(kind=kind, rows=_log(rng, 100, 2_000_000))
    if kind == "train":
        return dict(kind=kind, batch=32 * _log(rng, 2, 512), steps=rng.randint(1, 16))
    if kind == "maps":
        return dict(kind=kind, frames=rng.randint(1, 32), width=_log(rng, 60, 1100), height=_log(rng, 60, 1100), orient=rng.choice([8, 16, 32, 32]),
                    radius=rng.choice([3, 5, 8, 8, 8, 11]), half=rng.random() < 0.6)
    if kind == "volume":
        return dict(kind=kind, points=_log(rng, 2_000, 4_000_000), voxel=rng.uniform(0.0018, 0.008), weights=rng.random() < 0.7, tensor=rng.random() < 0.4)
    return dict(kind=kind, points=_log(rng, 200_000, 4_000_000), voxel=rng.uniform(0.003, 0.006), roots=_log(rng, 500, 20_000),
                stride=rng.randint(3, 6), batch=rng.choice([1024, 4096, 16_384]))


# ---- inputs: strands on a spherical scalp, cameras on an orbit, z-buffered maps -------------------------------------------------------


def _gen(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _u(g, n, lo=0.0, hi=1.0):
    return torch.rand(n, generator=g, device=DEV) * (hi - lo) + lo


def _unit(v):
    return v / v.norm(dim=-1, keepdim=True)


def _strands(g, n, hair, step=0.5e-3):
    """Strand vertices (n, J, 3), the tangent at each, and which are on a strand (lengths 60 to 150 mm)."""
    cz = _u(g, n, math.cos(math.radians(100.0)), 1.0)
    az, sz = _u(g, n, 0.0, 2 * math.pi), (1 - cz * cz).clamp_min(0).sqrt()
    out = torch.stack([sz * az.cos(), sz * az.sin(), cz], 1)
    fall = _unit(torch.stack([0.4 * az.cos(), 0.4 * az.sin(), -torch.ones_like(az)], 1))
    length, phase, which = _u(g, n, 0.06, 0.15), _u(g, n, 0.0, 2 * math.pi), _u(g, n)
    lo, hi, plo, phi = {"helix": (5e-3, 2e-2, 1e-2, 4e-2), "curls": (2e-3, 6e-3, 4e-3, 1e-2), "mixed": (5e-3, 1.5e-2, 2e-2, 6e-2)}[hair]
    r, pitch = _u(g, n, lo, hi), _u(g, n, plo, phi)
    wind = 2 * math.pi * r / pitch
    if hair == "mixed":  # half straight, half wavy
        r = torch.where(which < 0.5, torch.zeros_like(r), r)
        span = length / torch.where(which < 0.5, torch.ones_like(wind), (1 + 0.5 * wind * wind).sqrt())
    else:
        span = length / (1 + wind * wind).sqrt()
    j = torch.arange(int(math.ceil(0.15 / step)) + 1, device=DEV)
    s = (j[None, :] * step) / length[:, None] * span[:, None]  # along the centreline
    q = (s * s / (2 * span[:, None]))[..., None]
    side = _unit(torch.linalg.cross(out, fall))
    ang = (2 * math.pi / pitch)[:, None] * s + phase[:, None]
    x = SCALP * out[:, None, :] + out[:, None, :] * (s[..., None] - q) + fall[:, None, :] * q
    x = x + (r[:, None] * (ang.sin() - phase.sin()[:, None]))[..., None] * side[:, None, :]
    if hair != "mixed":
        other = torch.linalg.cross(_unit(out + fall), side)
        x = x + (r[:, None] * (ang.cos() - phase.cos()[:, None]))[..., None] * other[:, None, :]
    d = x[:, 1:] - x[:, :-1]
    on = (j[None, :-1] * step < length[:, None]).reshape(-1)
    return x[:, :-1].reshape(-1, 3)[on], _unit(d).reshape(-1, 3)[on], (torch.arange(n, device=DEV)[:, None].expand(-1, len(j) - 1).reshape(-1)[on])


def _cameras(views, width, height, arc):
    az = np.arange(views) * (360.0 / views) if arc >= 360 else np.linspace(-arc / 2, arc / 2, views)
    el, rec = math.radians(15.0), []
    for a in np.radians(az):
        c = 0.6 * np.array([math.cos(el) * math.cos(a), math.cos(el) * math.sin(a), math.sin(el)])
        f = -c / np.linalg.norm(c)
        rt = np.cross(f, [0.0, 0.0, 1.0])
        rt /= np.linalg.norm(rt)
        R = np.stack([rt, np.cross(f, rt), f])
        fl = width / (2.0 * math.tan(math.radians(25.0)))
        rec.append(np.concatenate([[fl, fl, (width - 1) / 2.0, (height - 1) / 2.0], R.ravel(), -R @ c]))
    return torch.from_numpy(np.stack(rec).astype(np.float32)).to(DEV)


def _project(cam, p):
    R, t = cam[4:13].reshape(3, 3), cam[13:16]
    x, y, z = (p[:, 0] * R[k, 0] + p[:, 1] * R[k, 1] + p[:, 2] * R[k, 2] + t[k] for k in range(3))
    return cam[0] * (x / z) + cam[2], cam[1] * (y / z) + cam[3], z


def _render(cam, x, d, width, height):
    """The strand vertex in front at each texel (-1: none), its image angle there, and the depth of strand or scalp (inf: neither)."""
    u, v, z = _project(cam, x)
    ix, iy = (u + 0.5).floor().long(), (v + 0.5).floor().long()
    ok = (z > 0.01) & (ix >= 0) & (ix < width) & (iy >= 0) & (iy < height)
    u2, v2, _ = _project(cam, x + 1e-3 * d)
    key = (z.contiguous().view(torch.int32).long() << 32) | torch.arange(len(x), device=DEV)
    none = torch.iinfo(torch.int64).max
    buf = torch.full((width * height + 1,), none, dtype=torch.int64, device=DEV)
    buf.scatter_reduce_(0, torch.where(ok, iy * width + ix, width * height), key, "amin")
    buf = buf[:-1]
    i = torch.where(buf == none, 0, buf & 0xFFFFFFFF)
    zs = torch.where(buf == none, math.inf, z[i])
    gx = (torch.arange(width, device=DEV) - cam[2]) / cam[0]
    gy = (torch.arange(height, device=DEV) - cam[3]) / cam[1]
    t = cam[13:16]
    dt, dd = gx[None, :] * t[0] + gy[:, None] * t[1] + t[2], gx[None, :] ** 2 + gy[:, None] ** 2 + 1
    disc = dt * dt - dd * ((t * t).sum() - SCALP * SCALP)
    zh = torch.where(disc > 0, (dt - disc.clamp_min(0).sqrt()) / dd, math.inf).reshape(-1)
    hair = zs <= zh
    ang = torch.remainder(torch.atan2((v2 - v)[i], (u2 - u)[i]), math.pi)
    return torch.where(hair & (buf != none), i, -1), ang, torch.minimum(zs, zh)


def _scene(case, seed, points, views, width, strands):
    g = _gen(seed)
    x, d, _ = _strands(g, strands, case["hair"])
    height = width
    cams = _cameras(views, width, height, case["arc"])
    dt = torch.float16 if case["half"] else torch.float32
    theta, conf, depth = (torch.empty((views, height, width), dtype=dt, device=DEV) for _ in range(3))
    for v in range(views):
        i, ang, z = _render(cams[v], x, d, width, height)
        n = width * height
        ang = ang + case["noise"] * torch.randn(n, generator=g, device=DEV)
        odd = _u(g, n) < case["outliers"]
        ang = torch.where(odd, _u(g, n, 0.0, math.pi), torch.remainder(ang, math.pi))
        c = torch.where(odd, _u(g, n), _u(g, n, 0.6, 1.0))
        theta[v] = torch.where(i >= 0, ang, 0.0).reshape(height, width).to(dt)
        conf[v] = torch.where(i >= 0, c, 0.0).reshape(height, width).to(dt)
        depth[v] = z.reshape(height, width).to(dt)
    # the outer layer: jittered strand points that at least two views see
    at = torch.randint(len(x), (4 * points,), generator=g, device=DEV)
    p = x[at] + 2e-3 * torch.randn((4 * points, 3), generator=g, device=DEV)
    seen = torch.zeros(4 * points, dtype=torch.int32, device=DEV)
    for v in range(views):
        u, w, z = _project(cams[v], p)
        ix, iy = (u + 0.5).floor().long(), (w + 0.5).floor().long()
        ok = (ix >= 0) & (ix < width) & (iy >= 0) & (iy < height)
        zd = depth[v][iy.clamp(0, height - 1), ix.clamp(0, width - 1)].float()
        seen += (ok & ((z - zd).abs() <= VIS_TAU)).int()
    keep = torch.argsort((seen < 2).int(), stable=True)[:points]
    return dict(points=p[keep].contiguous(), cams=cams, orient_maps=theta, conf_maps=conf, depth_maps=depth if case["depth"] else None)


def _rows(g, n):
    """Network inputs as a head gives them (8 to 16 views that see the point, the plane that each one's orientation spans) and the tangents."""
    t, out = _unit(torch.randn((n, 3), generator=g, device=DEV)), _unit(torch.randn((n, 3), generator=g, device=DEV))
    v = _unit(out[:, None, :] + 0.6 * torch.randn((n, 16, 3), generator=g, device=DEV))
    z = torch.zeros_like(v)
    z[..., 2] = 1.0
    e1 = _unit(torch.linalg.cross(z, v))
    e2 = torch.linalg.cross(v, e1)
    psi = torch.atan2((e2 * t[:, None]).sum(-1), (e1 * t[:, None]).sum(-1)) + 0.3 * torch.randn((n, 16), generator=g, device=DEV)
    c = torch.rand((n, 16), generator=g, device=DEV)
    m = c * (0.4 + 0.6 * torch.rand((n, 16), generator=g, device=DEV))
    f = torch.cat([(m * (2 * psi).cos())[..., None], (m * (2 * psi).sin())[..., None], c[..., None], v, torch.ones_like(c)[..., None]], -1)
    held = torch.randint(8, 17, (n, 1), generator=g, device=DEV) > torch.arange(16, device=DEV)[None]
    return (f * held[..., None]).reshape(n, 112).to(torch.bfloat16), t


def _hair_volume(g, points, strands):
    """Oriented points over the whole hair: tangents 10 degrees off, a tenth of them outliers, and how far each can be trusted."""
    x, d, _ = _strands(g, strands, "mixed")
    at = torch.randint(len(x), (points,), generator=g, device=DEV)
    p = x[at] + 2e-3 * torch.randn((points, 3), generator=g, device=DEV)
    odd = _u(g, points) < 0.1
    t = d[at] + math.radians(10.0) * torch.randn((points, 3), generator=g, device=DEV)
    t = _unit(torch.where(odd[:, None], torch.randn((points, 3), generator=g, device=DEV), t))
    return p.contiguous(), t.contiguous(), torch.where(odd, _u(g, points, 0.0, 0.5), _u(g, points, 0.5, 1.0))


def _grid(voxel):
    """A box around the hair; the few points that lie outside are not counted."""
    h = np.float32(voxel)
    origin = (np.floor(np.array([-0.19, -0.19, -0.22], np.float32) / h) * h).astype(np.float32)
    return origin, h, (np.ceil((np.array([0.19, 0.19, 0.20], np.float32) - origin) / h) + 1).astype(np.int32)


def _scene_sizes(case):
    """(points, views, resolution, strands) of each scene of a batch: `ratio` between the largest and the smallest."""
    n = case["scenes"]
    w = np.array([case["ratio"] ** (i / max(1, n - 1)) for i in range(n)])
    even = case["ratio"] == 1.0
    return [(max(1, int(case["points"] * w[i] / w.sum())), case["views"] if even else max(8, case["views"] * (1 + (3 * i) % 4) // 4),
             case["res"] if even else max(64, case["res"] * (2 + (7 * i) % 3) // 4), case["strands"]) for i in range(n)]


def prepare(case, seed):
    kind, g = case["kind"], _gen(seed)
    if kind in ("search", "features"):
        sc = _scene(case, seed, case["points"], case["views"], case["res"], case["strands"])
        if kind == "features":
            return dict(case=case, sc=sc)
        st = dict(case=case, sc=sc, kw=_search_args(case), ctx=native.Context(max_points=case["points"], max_views=case["views"]))
        if case["mode"] == "learned":
            st["net"] = native.MLP(path=WEIGHTS)
            st["kw"] |= _learned_args(st["net"])
        return st
    if kind == "batch":
        sizes = _scene_sizes(case)
        scenes = [_scene(case, seed + 1000 * i, *s) for i, s in enumerate(sizes)]
        for s in scenes:
            n = len(s["points"])
            s["dirs"], s["costs"] = torch.empty((n, 3), device=DEV), torch.empty(n, device=DEV)
        ctx = native.Context(max_points=sum(s[0] for s in sizes), max_views=sum(s[1] for s in sizes), max_scenes=len(sizes))
        if case["tuned"]:
            ctx.set_tuned(1, -1)
        st = dict(case=case, scenes=scenes, ctx=ctx, kw=_search_args(case))
        if case["mode"] == "learned":
            st["net"] = native.MLP(path=WEIGHTS)
            st["kw"] |= _learned_args(st["net"])
        return st
    if kind == "forward":
        return dict(case=case, net=native.MLP(path=WEIGHTS), feats=_rows(g, case["rows"])[0])
    if kind == "train":
        f, t = _rows(g, case["batch"] * case["steps"])
        return dict(case=case, net=native.MLP(path=WEIGHTS), feats=f.split(case["batch"]), targets=t.split(case["batch"]),
                    losses=torch.empty(case["steps"], device=DEV))
    if kind == "maps":
        x, d, sid = _strands(g, 4000, "mixed")
        cams = _cameras(case["frames"], case["width"], case["height"], 360)
        albedo = _u(g, 4000, 0.35, 1.0)
        frames = torch.empty((case["frames"], case["height"], case["width"]), device=DEV)
        for v in range(case["frames"]):
            i, _, z = _render(cams[v], x, d, case["width"], case["height"])
            grey = torch.where(i >= 0, albedo[sid[i.clamp_min(0)]], torch.where(torch.isfinite(z), 0.15, 0.0))
            frames[v] = (grey + 0.02 * torch.randn(len(grey), generator=g, device=DEV)).reshape(case["height"], case["width"])
        return dict(case=case, frames=frames, ctx=native.Context())
    p, d, w = _hair_volume(g, case["points"], 20_000)
    origin, h, dims = _grid(case["voxel"])
    ctx = native.Context()
    if kind == "volume":
        return dict(case=case, p=p, d=d, w=w if case["weights"] else None, grid=(origin, h, dims), ctx=ctx)
    occ, vd, vc = native.fuse_volume(p, d, origin, h, dims, weights=w, ctx=ctx)
    root = _unit(torch.stack([torch.randn(case["roots"], generator=g, device=DEV), torch.randn(case["roots"], generator=g, device=DEV),
                              torch.randn(case["roots"], generator=g, device=DEV).abs()], 1))
    ax = [torch.arange(0, int(n), case["stride"], device=DEV) for n in dims]
    iz, iy, ix = torch.meshgrid(ax[2], ax[1], ax[0], indexing="ij")
    seeds = torch.stack([ix, iy, iz], -1).reshape(-1, 3).float()
    seeds = torch.from_numpy(origin).to(DEV) + (seeds + 0.5) * float(h)
    return dict(case=case, volume=(occ, vd, vc), grid=(origin, h, dims), roots=(SCALP * root).contiguous(), normals=root.contiguous(),
                seeds=seeds.contiguous(), crossings=torch.zeros(int(np.prod(dims.astype(np.int64))), dtype=torch.int32, device=DEV),
                strands=torch.zeros((120 * case["roots"], 3), device=DEV), ctx=ctx)


def _search_args(case):
    mode = {"plain": native.FD_MODE_PLAIN, "learned": native.FD_MODE_LEARNED, "fpmvo": native.FD_MODE_FPMVO}[case["mode"]]
    return dict(patch=case["patch"], n_candidates=case["candidates"], refine_iters=case["iters"], top_k=case["top_k"], mode=mode)


def _learned_args(net):
    step0, tau = net.calibration()
    return dict(mlp=net, learned_iters=2, learned_step0=step0, fallback_cost=tau)


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "search":
        s = state["sc"]
        return native.fuse_directions(s["points"], s["cams"], s["orient_maps"], s["conf_maps"], depth_maps=s["depth_maps"], ctx=state["ctx"], **state["kw"])
    if kind == "features":
        s = state["sc"]
        return native.features(s["points"], s["cams"], s["orient_maps"], s["conf_maps"], depth_maps=s["depth_maps"])
    if kind == "batch":
        native.fuse_batched(state["scenes"], state["ctx"], **state["kw"])
        return [(s["dirs"], s["costs"]) for s in state["scenes"]]
    if kind == "forward":
        return state["net"].forward(state["feats"])
    if kind == "train":
        for k, (f, t) in enumerate(zip(state["feats"], state["targets"])):
            state["net"].train_step(f, t, lr=1e-4, loss=state["losses"][k:k + 1])
        return state["losses"], state["net"].get_params()
    if kind == "maps":
        return native.orientation_maps(state["frames"], n_orient=case["orient"], radius=case["radius"],
                                       out_dtype=torch.float16 if case["half"] else torch.float32, ctx=state["ctx"])
    if kind == "volume":
        return native.fuse_volume(state["p"], state["d"], *state["grid"], weights=state["w"], tensor=case["tensor"], ctx=state["ctx"])
    # hair growing: guide strands from the roots, segments both ways from the seeds, then linked and assembled
    vol, R, N, L, cr, ctx = (*state["volume"], *state["grid"]), state["roots"], state["normals"], state["seeds"], state["crossings"], state["ctx"]
    cr.zero_()
    g = native.grow_strands(*vol, R, N, crossings=cr, batch=case["batch"], ctx=ctx, **GROW)
    f = native.grow_strands(*vol, L, None, crossings=cr, batch=1 << 20, seed_mode=native.FD_SEED_AWAY, ctx=ctx, **GROW)
    b = native.grow_strands(*vol, L, None, crossings=cr, batch=1 << 20, seed_mode=native.FD_SEED_TOWARDS, ctx=ctx, **GROW)
    gn, fn, bn = g[1].long(), f[1].long(), b[1].long()
    ag, a_s = torch.arange(len(R), device=R.device), torch.arange(len(L), device=L.device)
    flags = torch.cat([(gn > 1).to(torch.uint8), ((fn > 1) & (bn > 1)).to(torch.uint8) * 3])
    succ = native.link_segments(torch.cat([R, b[0][a_s, bn - 1]]), torch.cat([N, b[2]]), torch.cat([g[0][ag, gn - 1], f[0][a_s, fn - 1]]),
                                torch.cat([g[2], f[2]]), flags, ctx=ctx, **LINK)
    return native.assemble_strands(g, f, b, succ, out=state["strands"], ctx=ctx) + (succ, cr)


# ---- what a pass cannot do without ----------------------------------------------------------------------------------------------------


def _search_work(case, points, views, width):
    size = 2 if case["half"] else 4
    # the maps, or the texels that the points' patches touch where that is less; points in, directions and costs out
    maps = views * width * width * size * (3 if case["depth"] else 2)
    touched = points * size * (case["top_k"] * (case["patch"] + 1) ** 2 * 2 + views * (1 if case["depth"] else 4))
    if case["mode"] == "fpmvo":
        evals = 5 * case["top_k"] * case["patch"] ** 2
    else:
        evals = (case["candidates"] + 6 * case["iters"]) * case["top_k"] * case["patch"] ** 2
    # 6 operations for a sample of one candidate in one view; the network's products where it runs
    return dict(bytes=min(maps, touched) + points * 28 + views * 64,
                flops=points * (6 * evals + 30 * views + (2 * 160512 if case["mode"] == "learned" else 0)))


def work(case):
    kind = case["kind"]
    if kind == "search":
        return _search_work(case, case["points"], case["views"], case["res"])
    if kind == "batch":
        each = [_search_work(case, p, v, r) for p, v, r, _ in _scene_sizes(case)]
        return {k: sum(e[k] for e in each) for k in ("bytes", "flops")}
    if kind == "features":
        size, n, v = 2 if case["half"] else 4, case["points"], case["views"]
        maps, touched = v * case["res"] ** 2 * size * (3 if case["depth"] else 2), n * size * (16 * 8 + (v if case["depth"] else 0))
        return dict(bytes=min(maps, touched) + n * (12 + 224), flops=n * (30 * v + 16 * 150))
    if kind == "forward":
        return dict(bytes=case["rows"] * (224 + 12) + 321_000, flops=case["rows"] * 2 * 160512)
    if kind == "train":
        # forward, weight gradients, input gradients of the last three layers; weights and moments in and out
        return dict(bytes=case["steps"] * (case["batch"] * 236 + 6 * 645_132), flops=case["steps"] * case["batch"] * 905_728)
    if kind == "maps":
        n = case["frames"] * case["width"] * case["height"]
        return dict(bytes=n * (4 + 2 * (2 if case["half"] else 4)), flops=n * 2 * case["orient"] * (2 * case["radius"] + 1) ** 2)
    if kind == "volume":
        nv = int(np.prod(_grid(case["voxel"])[2].astype(np.int64)))
        return dict(bytes=case["points"] * (24 + (4 if case["weights"] else 0)) + nv * (20 + (48 if case["tensor"] else 0)), flops=case["points"] * 30)
    # 1 mm steps: what a step reads of its voxel and the vertex that it writes (about 20 steps a trace)
    traces = case["roots"] + 2 * int(np.prod(-(-_grid(case["voxel"])[2].astype(np.int64) // case["stride"])))
    return dict(bytes=traces * 20 * 36, flops=traces * 20 * 40)


# ---- the same in 64 bits --------------------------------------------------------------------------------------------------------------


def _project64(cams, p):
    R, t = cams[:, 4:13].reshape(-1, 3, 3), cams[:, 13:16]
    c = [sum(p[:, a, None] * R[None, :, k, a] for a in range(3)) + t[None, :, k] for k in range(3)]
    return c[0], c[1], c[2], cams[None, :, 0] * (c[0] / c[2]) + cams[None, :, 2], cams[None, :, 1] * (c[1] / c[2]) + cams[None, :, 3]


def _texel(m, v, x, y):
    """m[v, y, x] in 64 bits, 0 outside."""
    _, H, W = m.shape
    ok = (x >= 0) & (x < W) & (y >= 0) & (y < H)
    return torch.where(ok, m.reshape(-1)[(v * H + y.clamp(0, H - 1)) * W + x.clamp(0, W - 1)].double(), 0.0)


def _sample(sc, v, u, w):
    """Bilinear confidence and confidence-weighted doubled-angle vector of view v at (u, w)."""
    x0, y0 = u.floor(), w.floor()
    fx, fy, ix, iy = u - x0, w - y0, x0.long(), y0.long()
    cb, mx, my = 0.0, 0.0, 0.0
    for b in (0, 1):
        for a in (0, 1):
            wt = (fx if a else 1 - fx) * (fy if b else 1 - fy)
            c = wt * _texel(sc["conf_maps"], v, ix + a, iy + b)
            t = 2 * _texel(sc["orient_maps"], v, ix + a, iy + b)
            cb, mx, my = cb + c, mx + c * t.cos(), my + c * t.sin()
    return cb, mx, my


def _eligible(sc, p, cams):
    X, Y, Z, u, w = _project64(cams, p)
    _, H, W = sc["conf_maps"].shape
    ok = (Z > 1e-3) & (u >= 0) & (u <= W - 1) & (w >= 0) & (w <= H - 1)
    views = torch.arange(len(cams), device=DEV)[None].expand(len(p), -1)
    if sc["depth_maps"] is not None:
        D = _texel(sc["depth_maps"], views, torch.where(ok, (u + 0.5).floor(), 0.0).long(), torch.where(ok, (w + 0.5).floor(), 0.0).long())
        ok = ok & ((Z - D).abs() <= np.float64(np.float32(VIS_TAU)))
    return ok, u, w, views


def _search64(case, sc, p):
    cams = sc["cams"].double()
    ok, u, w, views = _eligible(sc, p, cams)
    uu, ww = torch.where(ok, u, 0.0), torch.where(ok, w, 0.0)
    conf = torch.where(ok, _sample(sc, views, uu, ww)[0], 0.0)
    score, ids = torch.sort(conf, dim=1, descending=True, stable=True)
    K, h = case["top_k"], case["patch"] // 2
    on, ids = score[:, :K] > 0, ids[:, :K]
    keff = on.sum(1)
    cam = cams[ids]
    R, t = cam[..., 4:13].reshape(len(p), K, 3, 3), cam[..., 13:16]
    c = (R * p[:, None, None, :]).sum(-1) + t
    X, Y, Z = c.unbind(-1)
    u, w = cam[..., 0] * (X / Z) + cam[..., 2], cam[..., 1] * (Y / Z) + cam[..., 3]
    M = torch.stack([cam[..., 0, None] * (Z[..., None] * R[:, :, 0] - X[..., None] * R[:, :, 2]),
                     cam[..., 1, None] * (Z[..., None] * R[:, :, 1] - Y[..., None] * R[:, :, 2])], 2)
    A, B, C = [], [], []
    for b in range(-h, h + 1):
        for a in range(-h, h + 1):
            cb, mx, my = _sample(sc, ids, torch.where(on, u, 0.0) + a, torch.where(on, w, 0.0) + b)
            n = (mx * mx + my * my).sqrt()
            al = torch.where(on & (n > 0), 0.5 * cb * cb, 0.0)
            nn = torch.where(n > 0, n, 1.0)
            A.append(al), B.append(al * mx / nn), C.append(2 * al * my / nn)
    A, B, C = (torch.stack(v, -1) for v in (A, B, C))

    def S(d):  # view sum at a direction per point (n, 3)
        r = (M * d[:, None, None, :]).sum(-1)
        n2 = (r * r).sum(-1)
        nn = torch.where(n2 > 0, n2, 1.0)
        c2, s2 = (r[..., 0] ** 2 - r[..., 1] ** 2) / nn, r[..., 0] * r[..., 1] / nn
        q = (A + B * c2[..., None] + C * s2[..., None]).amax(-1)
        return torch.where(n2 > 0, q.clamp_min(0).sqrt(), 0.0).sum(1)

    return S, keff, (ids, on, u, w, Z, cam, R, score[:, :K])


def _flip(d):
    key = torch.where(d[:, 2] != 0, d[:, 2], torch.where(d[:, 1] != 0, d[:, 1], d[:, 0]))
    return torch.where((key < 0)[:, None], -d, d)


def _plain64(case, sc, p):
    S, keff, _ = _search64(case, sc, p)
    n = case["candidates"]
    k = np.arange(n, dtype=np.float64)
    z = 1 - (k + 0.5) / n
    rho, psi = np.sqrt(np.maximum(0, 1 - z * z)), k * math.pi * (3 - math.sqrt(5.0))
    lat = torch.from_numpy(np.stack([rho * np.cos(psi), rho * np.sin(psi), z], 1)).to(DEV)
    best, at = torch.full((len(p),), -math.inf, dtype=torch.float64, device=DEV), torch.zeros(len(p), dtype=torch.long, device=DEV)
    for i in range(n):
        s = S(lat[i][None].expand(len(p), 3))
        better = s > best
        best, at = torch.where(better, s, best), torch.where(better, i, at)
    d = lat[at]
    alpha = 0.5 * math.sqrt(2 * math.pi / n)
    for _ in range(case["iters"]):
        sg = torch.where(torch.signbit(d[:, 2]), -1.0, 1.0).double()
        a = -1 / (sg + d[:, 2])
        b = d[:, 0] * d[:, 1] * a
        e1 = torch.stack([1 + sg * d[:, 0] ** 2 * a, sg * b, -sg * d[:, 0]], 1)
        e2 = torch.stack([b, sg + d[:, 1] ** 2 * a, -d[:, 1]], 1)
        top, new = S(d), d
        for j in range(6):
            cand = math.cos(alpha) * d + math.sin(alpha) * (math.cos(j * math.pi / 3) * e1 + math.sin(j * math.pi / 3) * e2)
            s = S(cand)
            better = s > top
            top, new = torch.where(better, s, top), torch.where(better[:, None], cand, new)
        d, alpha = _unit(new), alpha / 2
    J = torch.where(keff > 0, 1 - S(d) / keff.clamp_min(1), math.inf)
    return torch.where((keff > 0)[:, None], _flip(d), 0.0), J


def _fpmvo64(case, sc, p):
    S, keff, (ids, on, u, w, Z, cam, R, score) = _search64(case, sc, p)
    _, H, W = sc["conf_maps"].shape
    cb, mx, my = _sample(sc, ids, torch.where(on, u, 0.0), torch.where(on, w, 0.0))
    t = 0.5 * torch.atan2(my, mx)
    ux, uy = u + 3.0 * t.cos(), w + 3.0 * t.sin()
    ok = on & ((mx * mx + my * my) > 0) & (ux >= 0) & (ux <= W - 1) & (uy >= 0) & (uy <= H - 1)
    D = _texel(sc["depth_maps"], ids, torch.where(ok, (ux + 0.5).floor(), 0.0).long(), torch.where(ok, (uy + 0.5).floor(), 0.0).long())
    ok = ok & torch.isfinite(D)
    delta = float(np.float32(5e-3))
    best = torch.full((len(p),), -math.inf, dtype=torch.float64, device=DEV)
    for s in range(5):
        z = torch.where(ok, D, 1.0) - delta + 2 * delta * s / 4
        c = torch.stack([(ux - cam[..., 2]) * z / cam[..., 0], (uy - cam[..., 3]) * z / cam[..., 1], z], -1) - cam[..., 13:16]
        d = (R * c[..., :, None]).sum(2) - p[:, None, :]
        n = d.norm(dim=-1)
        good = ok & (z > 0) & (n > 0)
        d = torch.where(good[..., None], d / torch.where(n > 0, n, 1.0)[..., None], 0.0)
        wt = torch.where(good, cb, 0.0)
        G = (d[:, :, None, :] * d[:, None, :, :]).sum(-1).abs()
        G = G * (1 - torch.eye(G.shape[1], device=DEV)) + torch.eye(G.shape[1], device=DEV)
        sigma = torch.where(good, (wt[:, None, :] * G).sum(-1) / wt.sum(-1, keepdim=True), -math.inf)
        f = d[torch.arange(len(p), device=DEV), sigma.argmax(1)]
        best = torch.where(good.any(1), torch.maximum(best, S(f)), best)
    # the directions are a choice among fused candidates that score alike: no 64-bit value of their own
    return None, torch.where((keff > 0) & torch.isfinite(best), 1 - best / keff.clamp_min(1), math.inf)


def _features64(sc, p):
    cams = sc["cams"].double()
    ok, u, w, views = _eligible(sc, p, cams)
    R, t = cams[:, 4:13].reshape(-1, 3, 3), cams[:, 13:16]
    centre = -(R * t[:, :, None]).sum(1)
    a = centre[None] - p[:, None]
    key = torch.where(ok, (a * p[:, None]).sum(-1) / a.norm(dim=-1), -math.inf)
    key, ids = torch.sort(key, dim=1, descending=True, stable=True)
    n = min(16, key.shape[1])
    on, ids = torch.isfinite(key[:, :n]), ids[:, :n]
    pick = lambda x: torch.where(on, x.gather(1, ids), 0.0)  # noqa: E731
    cb, mx, my = _sample(sc, ids, pick(u), pick(w))
    v = _unit(centre[ids] - p[:, None])
    cam, Rv = cams[ids], R[ids]
    c = (Rv * p[:, None, None, :]).sum(-1) + cam[..., 13:16]
    th = 0.5 * torch.atan2(my, mx)
    dl = torch.stack([th.cos() / cam[..., 0], th.sin() / cam[..., 1], torch.zeros_like(th)], -1)
    normal = (Rv * torch.linalg.cross(c, dl)[..., :, None]).sum(2)
    tt = torch.linalg.cross(normal, v)
    up = torch.zeros_like(v)
    up[..., 2] = 1.0
    e1 = _unit(torch.linalg.cross(up, v))
    psi = torch.atan2((tt * torch.linalg.cross(v, e1)).sum(-1), (tt * e1).sum(-1))
    m = (mx * mx + my * my).sqrt()
    f = torch.cat([(m * (2 * psi).cos())[..., None], (m * (2 * psi).sin())[..., None], cb[..., None], v, torch.ones_like(m)[..., None]], -1)
    full = torch.zeros((len(p), 16, 7), dtype=torch.float64, device=DEV)
    full[:, :n] = torch.where(on[..., None], f, 0.0)
    return full.reshape(len(p), 112)


def _weights():
    with open(WEIGHTS, "rb") as f:
        head, flat = f.read(48), np.frombuffer(f.read(), np.float32)
    n = len(flat) // 3
    return struct.unpack("<q", head[32:40])[0], [torch.from_numpy(flat[k * n:(k + 1) * n].astype(np.float64)).to(DEV) for k in range(3)]


def _layers(flat):
    at, got = 0, []
    for k, n in ((112, 256), (256, 256), (256, 256), (256, 3)):
        got.append((flat[at:at + k * n].reshape(k, n), flat[at + k * n:at + k * n + n]))
        at += k * n + n
    return got


def _network(flat, x):
    for i, (W, b) in enumerate(_layers(flat)):
        x = x @ W + b
        if i < 3:
            x = 0.5 * x * (1 + torch.tanh(math.sqrt(2 / math.pi) * (x + 0.044715 * x ** 3)))
    return _unit(x)


def _volume64(st):
    p, d, w, (origin, h, dims) = st["p"], st["d"].double(), st["w"], st["grid"]
    q = torch.floor((p - torch.from_numpy(origin).to(DEV)) / torch.tensor(h, device=DEV)).long()  # a whole number, taken in 32 bits by its rule
    nx, ny, nz = (int(v) for v in dims)
    nv = nx * ny * nz
    inside = ((q >= 0) & (q < torch.tensor([nx, ny, nz], device=DEV))).all(1)
    v = ((q[:, 2] * ny + q[:, 1]) * nx + q[:, 0])[inside]
    occ = torch.bincount(v, minlength=nv)
    wt = torch.ones(len(p), dtype=torch.float64, device=DEV) if w is None else w.double().clamp(0, 1)
    d, wt = d[inside], wt[inside]
    pairs = ((0, 0), (1, 1), (2, 2), (0, 1), (0, 2), (1, 2))
    T = torch.stack([torch.zeros(nv, dtype=torch.float64, device=DEV).index_add_(0, v, wt * d[:, a] * d[:, b]) for a, b in pairs], 1)
    busy = (T[:, :3].sum(1) > 0).nonzero()[:, 0]
    t = T[busy]
    A = {(0, 0): t[:, 0], (1, 1): t[:, 1], (2, 2): t[:, 2], (0, 1): t[:, 3], (0, 2): t[:, 4], (1, 2): t[:, 5]}
    get = lambda i, j: A[(min(i, j), max(i, j))]  # noqa: E731
    V = [[torch.full_like(t[:, 0], float(i == j)) for j in range(3)] for i in range(3)]
    for _ in range(12):  # cyclic Jacobi
        for a, b in ((0, 1), (0, 2), (1, 2)):
            k, apq = 3 - a - b, get(a, b)
            th = (A[(b, b)] - A[(a, a)]) / torch.where(apq != 0, 2 * apq, 1.0)
            tn = torch.where(apq != 0, torch.where(th >= 0, 1.0, -1.0) / (th.abs() + (th * th + 1).sqrt()), 0.0)
            c = 1 / (tn * tn + 1).sqrt()
            s = tn * c
            ka, kb = get(k, a), get(k, b)
            A[(a, a)], A[(b, b)], A[(a, b)] = A[(a, a)] - tn * apq, A[(b, b)] + tn * apq, torch.zeros_like(apq)
            A[(min(k, a), max(k, a))], A[(min(k, b), max(k, b))] = c * ka - s * kb, s * ka + c * kb
            for r in V:
                r[a], r[b] = c * r[a] - s * r[b], s * r[a] + c * r[b]
    lam, order = torch.sort(torch.stack([A[(i, i)] for i in range(3)], 1), dim=1, descending=True, stable=True)
    e = torch.stack([torch.stack(r, 1).gather(1, order[:, :1])[:, 0] for r in V], 1)
    dirs, coh = torch.zeros((nv, 3), dtype=torch.float64, device=DEV), torch.zeros(nv, dtype=torch.float64, device=DEV)
    dirs[busy], coh[busy] = _flip(_unit(e)), (lam[:, 0] - lam[:, 1]) / lam[:, 0]
    shape = (nz, ny, nx)
    out = (occ.int().reshape(shape), dirs.reshape(shape + (3,)), coh.reshape(shape))
    return out + (T.reshape(shape + (6,)),) if st["case"]["tensor"] else out


def _maps64(st):
    case, frames = st["case"], st["frames"]
    N, R = case["orient"], case["radius"]
    th = torch.arange(N, dtype=torch.float64, device=DEV) * math.pi / N
    ax = torch.arange(-R, R + 1, dtype=torch.float64, device=DEV)
    dy, dx = torch.meshgrid(ax, ax, indexing="ij")
    a = dx * th.cos()[:, None, None] + dy * th.sin()[:, None, None]
    b = -dx * th.sin()[:, None, None] + dy * th.cos()[:, None, None]
    sa, sb = float(np.float32(2.4)), float(np.float32(1.8))
    bank = torch.exp(-a * a / (2 * sa * sa) - b * b / (2 * sb * sb)) * torch.cos(2 * math.pi * b / 4.0)
    bank = bank - bank.mean((1, 2), keepdim=True)
    k = torch.arange(N, device=DEV)
    apart = (k[:, None] - k[None]).abs()
    d2 = (torch.minimum(apart, N - apart) * (math.pi / N)).double() ** 2
    theta, conf = [], []
    H, W = frames.shape[1:]
    for f in frames:
        pad = torch.nn.functional.pad(f.double(), (R, R, R, R))
        F = torch.zeros((H * W, N), dtype=torch.float64, device=DEV)
        for i in range(2 * R + 1):  # a row of taps at a time
            win = pad[i:i + H].unfold(1, 2 * R + 1, 1).reshape(H * W, 2 * R + 1)
            F += win @ bank[:, i].T
        F = F.abs()
        top, j = F.max(1)
        c = (d2[j] * (F - top[:, None]) ** 2).sum(1).sqrt()
        theta.append((j * (math.pi / N)).double().reshape(H, W))
        conf.append((c / c.max() if c.max() > 0 else c).reshape(H, W))
    return torch.stack(theta), torch.stack(conf)


def _in_parts(fn, p, part):
    got = [fn(q.double()) for q in p.split(part)]
    if isinstance(got[0], tuple):
        return tuple(None if v[0] is None else torch.cat(v) for v in zip(*got))
    return torch.cat(got)


def exact(case, seed):
    kind = case["kind"]
    if kind == "strands" or case.get("mode") == "learned":
        # a trace is defined by its 32-bit steps, and the learned form keeps or drops a point by what a 16-bit network proposes: neither has a
        # value in 64 bits
        return None
    st = prepare(case, seed)
    if kind == "search":
        one = _plain64 if case["mode"] == "plain" else _fpmvo64
        return _in_parts(lambda q: one(case, st["sc"], q), st["sc"]["points"], max(256, 4_000_000 // (case["top_k"] * case["patch"] ** 2)))
    if kind == "batch":
        return [_in_parts(lambda q: _plain64(case, s, q), s["points"], max(256, 4_000_000 // (case["top_k"] * case["patch"] ** 2)))
                for s in st["scenes"]]
    if kind == "features":
        return _in_parts(lambda q: _features64(st["sc"], q), st["sc"]["points"], 20_000)
    if kind == "forward":
        flat = _weights()[1][0]
        return torch.cat([_network(flat, x.double()) for x in st["feats"].split(200_000)])
    if kind == "train":
        step, (w, m, v) = _weights()
        losses = []
        for f, t in zip(st["feats"], st["targets"]):
            w = w.detach().requires_grad_()
            loss = (1 - (_network(w, f.double()) * t.double()).sum(1) ** 2).mean()
            (gr,) = torch.autograd.grad(loss, w)
            step += 1
            m, v = 0.9 * m + 0.1 * gr, 0.999 * v + 0.001 * gr * gr
            w = w.detach() - 1e-4 * (m / (1 - 0.9 ** step)) / ((v / (1 - 0.999 ** step)).sqrt() + 1e-8)
            losses.append(loss.detach())
        return torch.stack(losses), w
    return _maps64(st) if kind == "maps" else _volume64(st)
