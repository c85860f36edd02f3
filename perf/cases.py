"""What a user of this library has it do, as cases to time and compare: ray
queries, acceleration-structure builds and refits, the Stage-0 and
single-bounce reconstruction steps, light baking, and path tracing with and
without emitter sampling, over the sizes of the library's configurations and
the smaller ones around them.

Scenes are the benchmark's stand-ins drawn on the GPU: a cloud of random
surfels ("cloud"), an axis-aligned furnished room tiled with coplanar surfels
("room"), and the same room with every centre, quaternion and scale perturbed,
as a scene under optimisation has them ("worn"). `exact` is the method in
64-bit torch by brute force over all surfels.
"""
import math

import torch

from paper_2601_23065_amd import api

DEV = "cuda"
GRADS = ("pos", "rot", "scale", "opacity", "albedo", "radiance")
JITTER = 1


# ---------------------------------------------------------------------------
# the cases
# ---------------------------------------------------------------------------
def listed():
    return [
        # the smallest ray query: a probe of a small model, where launches and one ray's latency count
        dict(name="trace_cloud", kind="trace", scene="cloud", n=2000, rays=256, hits=0),
        # a batch of incoherent rays with their blended hit lists, an odd count, on a scene under optimisation
        dict(name="trace_room_hits", kind="trace", scene="worn", n=100_000, rays=30_011, hits=64),
        # building the tree of a small model, then a first query
        dict(name="build_cloud", kind="build", scene="cloud", n=2000, rays=256),
        # building the tree of the full-size room, then a first query
        dict(name="build_1m", kind="build", scene="room", n=1_000_000, rays=1021),
        # interactive edit: select a box, move it, update the tree, preview the 0-bounce image
        dict(name="edit_200k", kind="edit", scene="worn", n=200_000, width=160, height=120),
        # single-bounce reconstruction step on the small model, forward and backward
        dict(name="sb_cloud", kind="sb", scene="cloud", n=2000, width=64, height=64, cams=1, spp=4),
        # the reconstruction step at the size of its configuration
        dict(name="sb_100k", kind="sb", scene="room", n=100_000, width=256, height=256, cams=8, spp=8),
        # Stage-0 step on a scene under optimisation: images, objective, adjoint
        dict(name="stage0_100k", kind="stage0", scene="worn", n=100_000, width=256, height=256, cams=8),
        # one light-baking iteration on the full-size room
        dict(name="bake_1m", kind="bake", scene="room", n=1_000_000, width=512, height=384, cams=8),
        # a jittered preview frame at a ragged size
        dict(name="pt_preview", kind="pt", scene="room", n=20_000, width=187, height=101, spp=1, depth=5, rr=3,
             jitter=True),
        # a progressive pass of the full-size frame (the headline workload at a quarter of its samples)
        dict(name="pt_1m", kind="pt", scene="room", n=1_000_000, width=1024, height=768, spp=16, depth=5, rr=3,
             jitter=False),
        # a frame with emitter sampling by 1 m cells
        dict(name="mis_300k", kind="mis", scene="room", n=300_000, width=512, height=384, spp=4, depth=5, rr=3,
             cell=1.0),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["trace", "build", "edit", "sb", "stage0", "bake", "pt", "mis"])
    scene = rng.choice(["room", "worn", "cloud"])
    n = _log_int(rng, 2000, 8000) if scene == "cloud" else _log_int(rng, 10_000, 1_000_000)
    w, h = _log_int(rng, 40, 640), _log_int(rng, 40, 480)
    c = dict(kind=kind, scene=scene, n=n)
    if kind == "trace":
        return dict(c, rays=_log_int(rng, 100, 300_000), hits=rng.choice([0, 0, 16, 64]))
    if kind == "build":
        return dict(c, rays=_log_int(rng, 100, 2000))
    if kind == "edit":
        return dict(c, width=_log_int(rng, 40, 320), height=_log_int(rng, 40, 240))
    if kind in ("sb", "stage0", "bake"):
        c = dict(c, width=min(w, 256), height=min(h, 256), cams=rng.randint(1, 9))
        return dict(c, spp=rng.randint(1, 8)) if kind == "sb" else c
    c = dict(c, width=w, height=h, spp=rng.randint(1, 8), depth=rng.randint(1, 8), rr=rng.choice([0, 2, 3]))
    if kind == "pt":
        return dict(c, jitter=rng.random() < 0.5)
    return dict(c, cell=rng.choice([0.0, 1.0]))


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
class _Cam:
    def __init__(self, eye, look_at, up, width, height, vfov=60.0):
        self.eye, self.look_at, self.up = eye, look_at, up
        self.vfov_deg, self.width, self.height = vfov, width, height


def _uniform(g, lo, hi, *shape):
    return lo + (hi - lo) * torch.rand(*shape, generator=g, device=DEV, dtype=torch.float64)


def _cloud(n, g):
    q = torch.randn(4, n, generator=g, device=DEV, dtype=torch.float64)
    em = torch.rand(n, generator=g, device=DEV) < 0.01
    em[0] = True
    return dict(pos=_uniform(g, -1, 1, 3, n), rot=q / q.norm(dim=0),
                scale=torch.exp(_uniform(g, math.log(0.02), math.log(0.1), 2, n)), opacity=_uniform(g, 0.5, 0.99, n),
                albedo=_uniform(g, 0.1, 0.8, 3, n), radiance=_uniform(g, 1, 10, 3, n) * em, emissive=em.double())


# quaternions (w, x, y, z) that turn +z into each axis direction
_S = math.sqrt(0.5)
_TURN = {(0, 0, 1): (1, 0, 0, 0), (0, 0, -1): (0, 1, 0, 0), (1, 0, 0): (_S, 0, _S, 0), (-1, 0, 0): (_S, 0, -_S, 0),
         (0, 1, 0): (_S, -_S, 0, 0), (0, -1, 0): (_S, _S, 0, 0)}


def _box_faces(lo, hi, sign, skip_bottom=False):
    """(plane axis, its coordinate, lo, hi, normal) of a box's faces; sign +1 outward, -1 inward."""
    out = []
    for a in range(3):
        for hi_side in (0, 1):
            if skip_bottom and a == 2 and not hi_side:
                continue
            nrm = [0, 0, 0]
            nrm[a] = sign if hi_side else -sign
            out.append((a, (hi if hi_side else lo)[a], lo, hi, tuple(nrm)))
    return out


def _room(n, g, worn):
    size = (6.0, 4.0, 3.0) if n <= 300_000 else (8.0, 6.0, 3.0)
    faces = _box_faces((0.0, 0.0, 0.0), size, -1)
    furniture = torch.rand(12 if n <= 300_000 else 40, 5, generator=g, device=DEV, dtype=torch.float64).tolist()
    for a, b, c, d, e in furniture:
        w, dep, hgt = 0.4 + 1.2 * a, 0.4 + 1.2 * b, 0.4 + 0.8 * c
        x, y = 0.3 + d * (size[0] - 0.6 - w), 0.3 + e * (size[1] - 0.6 - dep)
        faces += _box_faces((x, y, 0.0), (x + w, y + dep, hgt), 1, skip_bottom=True)
    areas = []
    for a, _, lo, hi, _ in faces:
        e = [hi[k] - lo[k] for k in range(3) if k != a]
        areas.append(e[0] * e[1])
    n_em = max(1, n // 200)
    panels = max(1, round(n_em * 0.0175 / 10.0 / 0.72))
    cols = max(1, math.ceil(math.sqrt(panels * size[0] / size[1])))
    rows = math.ceil(panels / cols)
    lights = []
    for k in range(panels):
        x, y = (k % cols + 0.5) * size[0] / cols, (k // cols + 0.5) * size[1] / rows
        lights.append((2, size[2] - 0.01, (x - 0.6, y - 0.3, 0.0), (x + 0.6, y + 0.3, 0.0), (0, 0, -1)))
    pick = torch.cat([torch.multinomial(torch.tensor(areas, device=DEV), n - n_em, True, generator=g),
                      len(faces) + torch.randint(panels, (n_em,), generator=g, device=DEV)])
    faces += lights
    f64 = dict(device=DEV, dtype=torch.float64)
    lo, hi = torch.tensor([f[2] for f in faces], **f64).T[:, pick], torch.tensor([f[3] for f in faces], **f64).T[:, pick]
    pos = lo + (hi - lo) * torch.rand(3, n, generator=g, **f64)
    axis, plane = torch.tensor([f[0] for f in faces], device=DEV)[pick], torch.tensor([f[1] for f in faces], **f64)[pick]
    pos = torch.where(torch.arange(3, device=DEV)[:, None] == axis, plane, pos)
    half = _uniform(g, 0, math.pi, n)
    t = torch.tensor([_TURN[f[4]] for f in faces], **f64).T[:, pick]
    c, s = half.cos(), half.sin()
    rot = torch.stack([t[0] * c - t[3] * s, t[1] * c + t[2] * s, t[2] * c - t[1] * s, t[3] * c + t[0] * s])
    em = torch.arange(n, device=DEV) >= n - n_em
    sc = dict(pos=pos, rot=rot, scale=torch.exp(_uniform(g, math.log(0.01), math.log(0.05), 2, n)),
              opacity=_uniform(g, 0.6, 0.99, n), albedo=_uniform(g, 0.05, 0.9, 3, n),
              radiance=_uniform(g, 5, 20, n) * em * torch.ones(3, 1, **f64), emissive=em.double())
    if worn:
        sc["pos"] = sc["pos"] + 0.01 * torch.randn(3, n, generator=g, **f64)
        sc["rot"] = sc["rot"] + 0.01 * torch.randn(4, n, generator=g, **f64)
        sc["scale"] = sc["scale"] * torch.exp(0.01 * torch.randn(2, n, generator=g, **f64))
        # a radiance cache on every surfel, as the reconstruction stages keep one
        sc["radiance"] = sc["radiance"] + _uniform(g, 0, 2, 3, n)
    order = torch.randperm(n, generator=g, device=DEV)   # indices carry no face grouping
    return {k: v[..., order] for k, v in sc.items()}, size


def _scene(case, g):
    if case["scene"] == "cloud":
        arrays, size = _cloud(case["n"], g), None
    else:
        arrays, size = _room(case["n"], g, case["scene"] == "worn")
    return {k: v.float().contiguous() for k, v in arrays.items()}, size


def _cams(case, size, g):
    out = []
    for _ in range(case.get("cams", 1)):
        a, b, c, d, e = torch.rand(5, generator=g, device=DEV, dtype=torch.float64).tolist()
        yaw, pitch = 2 * math.pi * d, 0.26 * (2 * e - 1)
        v = (math.cos(pitch) * math.cos(yaw), math.cos(pitch) * math.sin(yaw), math.sin(pitch))
        if size is None:
            eye, at = tuple(-3 * x for x in v), (0.0, 0.0, 0.0)
        else:
            eye = (0.5 + a * (size[0] - 1), 0.5 + b * (size[1] - 1), 1.3 + 0.7 * c)
            at = tuple(x + y for x, y in zip(eye, v))
        out.append(_Cam(eye, at, (0.0, 0.0, 1.0), case["width"], case["height"]))
    return out


def _rays(case, size, g):
    m = case["rays"]
    d = torch.randn(3, m, generator=g, device=DEV, dtype=torch.float64)
    d = d / d.norm(dim=0)
    if size is None:
        o = -3 * d + 0.6 * (torch.rand(3, m, generator=g, device=DEV, dtype=torch.float64) - 0.5)
    else:
        o = 0.05 + torch.rand(3, m, generator=g, device=DEV, dtype=torch.float64) * \
            (torch.tensor(size, device=DEV, dtype=torch.float64)[:, None] - 0.1)
    return o.contiguous(), d.contiguous()


def _params(case, seed):
    if case["kind"] in ("pt", "mis"):
        return api.Params(spp=case["spp"], max_depth=case["depth"], rr_start=case["rr"], seed=seed,
                          flags=JITTER if case.get("jitter") else 0)
    return api.Params(spp=case.get("spp", 1), seed=seed)


def _inputs(case, seed):
    """Everything the seed decides: scene arrays, cameras or rays, targets."""
    g = torch.Generator(device=DEV).manual_seed(seed)
    arrays, size = _scene(case, g)
    s = dict(kind=case["kind"], arrays=arrays, params=_params(case, seed), hits=case.get("hits", 0))
    if "rays" in case:
        s["rays"] = _rays(case, size, g)
    else:
        s["cams"] = _cams(case, size, g)
    px = (case.get("cams", 1), case.get("height", 0), case.get("width", 0))
    if case["kind"] in ("sb", "stage0", "bake"):
        s["target"] = 2 * torch.rand(*px, 3, generator=g, device=DEV)
    if case["kind"] == "stage0":
        nm = torch.randn(*px, 3, generator=g, device=DEV)
        s["normal"] = nm / nm.norm(dim=-1, keepdim=True)
        s["mask"] = (torch.rand(*px, generator=g, device=DEV) < 0.05).float()
    if case["kind"] == "edit":
        lo = (-1.0, -1.0, -1.0) if size is None else (0.0, 0.0, 0.0)
        hi = (0.0, 0.0, 0.0) if size is None else (2.5, 2.5, 2.0)
        a = 0.2 + 0.1 * torch.rand(1, generator=g, device=DEV).item()
        s["edit"] = (lo, hi, (math.cos(a), 0.0, 0.0, math.sin(a)), (1.0, 1.0, 0.5), (0.4, 0.3, 0.0))
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    scene = s["scene"] = api.Scene({k: v.clone() for k, v in s["arrays"].items()})
    if s["kind"] != "build":
        s["bvh"] = api.BVH(scene)
    if s["kind"] == "sb":
        s["leaves"] = {k: scene.t[k].detach().requires_grad_() for k in GRADS}
    if s["kind"] == "bake":
        s["baker"] = api.Baker(s["bvh"], scene, s["cams"], s["params"], s["target"], api.Adam(lr=0.05))
    if s["kind"] == "pt":
        s["ws"] = api.path_trace_workspace(scene)
    if s["kind"] == "mis":
        s["emitters"] = api.Emitters(scene, s["params"], cell=case["cell"])
        s["ws"] = api.path_trace_mis_workspace(scene, s["cams"][0], s["params"])
    return s


def run(s):
    kind, scene, p, bvh = s["kind"], s["scene"], s["params"], s.get("bvh")
    if kind == "trace":
        return api.trace_rays(bvh, scene, p, *s["rays"], max_hits=s["hits"])
    if kind == "build":
        return api.trace_rays(api.BVH(scene), scene, p, *s["rays"])
    if kind == "edit":
        lo, hi, r, pivot, t = s["edit"]
        for k in ("pos", "rot"):
            scene.t[k].copy_(s["arrays"][k])
        idx = api.select_box(scene, lo, hi)
        api.move_surfels(scene, idx, r, pivot, t)
        s["bvh"], _ = api.update_bvh(bvh, scene)
        return scene.t["pos"], scene.t["rot"], api.render_zero_bounce(s["bvh"], scene, s["cams"], p)
    if kind == "sb":
        for v in s["leaves"].values():
            v.grad = None
        rgb = api.SingleBounceRender.apply(*s["leaves"].values(), scene.t["emissive"], bvh, scene, s["cams"], p)
        (rgb - s["target"]).square().mean().backward()
        return rgb.detach(), {k: v.grad for k, v in s["leaves"].items()}
    if kind == "stage0":
        images, state = api.render_stage0(bvh, scene, s["cams"], p)
        loss, d = api.stage0_loss(images, s["target"], s["normal"], s["mask"], s["cams"], p)
        return images, loss, api.stage0_backward(bvh, scene, s["cams"], p, d, state)
    if kind == "bake":
        b = s["baker"]
        return b.step(), scene.t["radiance"], b.m, b.v
    if kind == "pt":
        acc = api.path_trace(bvh, scene, s["cams"][0], p, ws=s["ws"])
    else:
        acc = api.path_trace_mis(bvh, scene, s["emitters"], s["cams"][0], p, ws=s["ws"])
    return api.resolve(acc, p.spp)


# Floors: the scene read once (68 B a surfel), inputs and outputs once, and
# about 100 operations for each blended hit (distance, ellipse coordinates,
# response, and the blend of 11 quantities).
_HITS = {"cloud": 12, "room": 40, "worn": 40}


def _segments(case):
    kind = case["kind"]
    if kind in ("trace", "build"):
        return case["rays"]
    px = case["width"] * case["height"] * case.get("cams", 1)
    if kind == "sb":
        return 2 * px * (1 + case["spp"])
    if kind in ("stage0", "bake"):
        return 2 * px
    if kind == "edit":
        return px
    return px * case["spp"] * min(1 + case["depth"], 3) * (2 if kind == "mis" else 1)


def work(case):
    n, kind, seg = case["n"], case["kind"], _segments(case)
    px = case.get("width", 0) * case.get("height", 0) * case.get("cams", 1)
    io = {"trace": 96 * seg + 4 * seg * case.get("hits", 0), "build": 96 * seg, "edit": 12 * px + 84 * n,
          "sb": 24 * px + 64 * n, "stage0": 100 * px + 56 * n, "bake": 24 * px + 36 * n}.get(kind, 36 * px)
    return dict(bytes=68.0 * n + io, flops=100.0 * _HITS[case["scene"]] * seg)


# ---------------------------------------------------------------------------
# the method in 64 bits, by brute force
# ---------------------------------------------------------------------------
def _frames(sc):
    w, x, y, z = sc["rot"] / sc["rot"].norm(dim=0)
    tu = torch.stack([1 - 2 * (y * y + z * z), 2 * (x * y + w * z), 2 * (x * z - w * y)])
    tv = torch.stack([2 * (x * y - w * z), 1 - 2 * (x * x + z * z), 2 * (y * z + w * x)])
    return tu, tv, torch.linalg.cross(tu, tv, dim=0)


def _cross(a, b):
    return torch.linalg.cross(a, b, dim=0)


def _hit_lists(sc, O, W, p):
    """Every hit of the rays O, W [3, m] in blending order: indices [m, k] and which of them are hits."""
    n, m = sc["opacity"].numel(), O.shape[1]
    tu, tv, nn = _frames(sc)
    pn, pu, pv = ((sc["pos"] * a).sum(0) for a in (nn, tu, tv))
    step = max(1, 100_000_000 // n)
    ray, idx, key = [], [], []
    for a in range(0, m, step):
        o, w = O[:, a:a + step].T.contiguous(), W[:, a:a + step].T.contiguous()
        den = w @ nn
        t = (pn - o @ nn) / den
        r = ((o @ tu + t * (w @ tu) - pu) / sc["scale"][0]) ** 2
        r += ((o @ tv + t * (w @ tv) - pv) / sc["scale"][1]) ** 2
        hit = (den.abs() > 1e-12) & (t > float(torch.tensor(p.t_min))) & (r <= p.k_sigma ** 2) & (sc["opacity"] > 0)
        i, j = hit.nonzero(as_tuple=True)
        ray.append(i + a)
        idx.append(j)
        key.append(torch.floor(t[i, j] / p.depth_quantum).long() * n + j)
    ray, idx, key = torch.cat(ray), torch.cat(idx), torch.cat(key)
    order = key.argsort(stable=True)
    order = order[ray[order].argsort(stable=True)]
    ray, idx = ray[order], idx[order]
    count = torch.bincount(ray, minlength=m)
    at = torch.arange(ray.numel(), device=DEV) - (count.cumsum(0) - count)[ray]
    k = max(1, int(count.max()))
    lists = torch.zeros(m, k, dtype=torch.long, device=DEV)
    lists[ray, at] = idx
    return lists, torch.arange(k, device=DEV) < count[:, None]


def _trace(sc, O, W, p):
    """(N, D, R, E, P, A, hit lists, blended mask) of the rays, differentiable in sc, O and W."""
    with torch.no_grad():
        lists, on = _hit_lists(sc, O, W, p)
    f = _frames(sc)
    tu, tv, nn = (a[:, lists] for a in f)
    pos, scale = sc["pos"][:, lists], sc["scale"][:, lists]
    o, w = O[:, :, None], W[:, :, None]
    den = (w * nn).sum(0)
    t = ((pos - o) * nn).sum(0) / torch.where(on, den, 1.0)
    y = o + t * w - pos
    r = ((y * tu).sum(0) / scale[0]) ** 2 + ((y * tv).sum(0) / scale[1]) ** 2
    alpha = torch.where(on, sc["opacity"][lists] * torch.exp(-0.5 * r), 0.0)
    after = torch.cumprod(1 - alpha, 1)
    before = torch.cat([torch.ones_like(after[:, :1]), after[:, :-1]], 1)
    on = on & ~(before.detach() < float(torch.tensor(p.T_min)))
    wt = torch.where(on, before * alpha, 0.0)
    N = (wt * torch.where(den > 0, -nn, nn)).sum(2)
    D = (wt * torch.where(on, t, 0.0)).sum(1)
    R, P = ((wt * sc[k][:, lists]).sum(2) for k in ("radiance", "albedo"))
    A = 1 - torch.where(on, 1 - alpha, 1.0).prod(1)
    return N, D, R, (wt * sc["emissive"][lists]).sum(1), P, A, lists, on


def _parts(total, sc):
    """Slices of a long list of rays that fit memory."""
    step = 1 << 15
    return [slice(a, min(total, a + step)) for a in range(0, total, step)]


def _camera(cam):
    e, at, up = (torch.tensor(v, dtype=torch.float32).double() for v in (cam.eye, cam.look_at, cam.up))
    f = at - e
    f = f / f.norm()
    r = torch.linalg.cross(f, up)
    r = r / r.norm()
    th = math.tan(math.radians(float(torch.tensor(cam.vfov_deg))) / 2)
    return e.to(DEV), (r * th * cam.width / cam.height).to(DEV), (torch.linalg.cross(r, f) * th).to(DEV), f.to(DEV)


def _pixel_rays(cam, pix, ox=0.5, oy=0.5):
    e, r, u, f = _camera(cam)
    dx = 2 * ((pix % cam.width) + ox) / cam.width - 1
    dy = 1 - 2 * ((pix // cam.width) + oy) / cam.height
    d = r[:, None] * dx + u[:, None] * dy + f[:, None]
    return e[:, None].expand_as(d), d / d.norm(dim=0)


def _philox(c0, c1, c2, c3, seed):
    """Uniforms in [0, 1) of the four words of Philox4x32-10 (24 bits of each)."""
    mask = 0xFFFFFFFF
    c = [torch.as_tensor(v, device=DEV, dtype=torch.long) + torch.zeros_like(c0) for v in (c0, c1, c2, c3)]
    k0, k1 = seed & mask, seed >> 32
    for _ in range(10):
        a, b = c[0] * 0xD2511F53, c[2] * 0xCD9E8D57
        c = [((b >> 32) & mask) ^ c[1] ^ k0, b & mask, ((a >> 32) & mask) ^ c[3] ^ k1, a & mask]
        k0, k1 = (k0 + 0x9E3779B9) & mask, (k1 + 0xBB67AE85) & mask
    return [(v >> 8).double() / 2.0 ** 24 for v in c]


def _bounce(N, u0, u1):
    h = torch.tensor([1.0, 2.0, 3.0], device=DEV, dtype=torch.float64)[:, None] / math.sqrt(14)
    b = h - (h * N).sum(0) * N
    b = b / b.norm(dim=0)
    r, phi = u0.sqrt(), 2 * math.pi * u1
    return r * phi.cos() * b + r * phi.sin() * _cross(N, b) + (1 - u0).sqrt() * N


def _tau(p):
    return float(torch.tensor(p.tau_E))


def _pq(x):
    ym = (x.clamp(min=0) / 10000) ** (2610 / 16384)
    return ((3424 / 4096 + 2413 / 128 * ym) / (1 + 2392 / 128 * ym)) ** (2523 / 32)


def _pq_slope(x):
    y = (x / 10000).clamp(min=2.0 ** -24)
    with torch.enable_grad():
        z = (10000 * y).detach().requires_grad_()
        (g,) = torch.autograd.grad(_pq(z).sum(), z)
    return torch.where(x < 0, 0.0, g)


def _exact_probe(sc, rays, p, max_hits):
    N, D, R, E, P, A, lists, on = _trace(sc, *rays, p)
    hit = on.any(1)
    unit = torch.where(hit, N / N.norm(dim=0).clamp(min=1e-300), 0.0)
    out = torch.cat([unit, torch.where(hit, D / A.clamp(min=1e-300), 0.0)[None], R, E[None], P, A[None]])
    return (out, None, None) if max_hits else out


def _exact_zero_bounce(sc, cams, p):
    px = torch.arange(cams[0].width * cams[0].height, device=DEV)
    img = [torch.cat([_trace(sc, *_pixel_rays(c, px[q]), p)[2] for q in _parts(px.numel(), sc)], 1).T for c in cams]
    return torch.stack(img).reshape(len(cams), cams[0].height, cams[0].width, 3)


def _exact_sb(sc, s):
    p, cams = s["params"], s["cams"]
    sc = {k: v.requires_grad_(k in GRADS) for k, v in sc.items()}
    target = s["target"].double()
    rgb, hw = torch.zeros_like(target), cams[0].width * cams[0].height
    for ci, cam in enumerate(cams):
        for a in range(0, hw, 4096):
            pix = torch.arange(a, min(hw, a + 4096), device=DEV)
            O, W = _pixel_rays(cam, pix)
            N, D, R, E, P, A, _, on = _trace(sc, O, W, p)
            hit = on.any(1)
            bounce = hit & ~(E > _tau(p))
            j = bounce.nonzero()[:, 0]
            X = (O + torch.where(hit, D / torch.where(hit, A, 1.0), 0.0) * W)[:, j]
            Nt = N[:, j] / N[:, j].norm(dim=0)
            mean = 0
            for k in range(p.spp):
                u = _philox(pix[j], k, 0, p.camera_id + ci, p.seed)
                mean = mean + _trace(sc, X, _bounce(Nt, u[0], u[1]), p)[2] / p.spp
            L = torch.where((hit & ~bounce)[:, None], R.T, 0.0).index_put((j,), (P[:, j] * mean).T)
            t = target[ci].reshape(-1, 3)[pix]
            ((L - t).square().sum() / target.numel()).backward()
            rgb[ci].reshape(-1, 3)[pix] = L.detach()
    return rgb, {k: sc[k].grad for k in GRADS}


def _exact_stage0(sc, s):
    p, cams = s["params"], s["cams"]
    W_, H_ = cams[0].width, cams[0].height
    px = torch.arange(W_ * H_, device=DEV)
    images, dirs = [], []
    for c in cams:
        rows = []
        for q in _parts(px.numel(), sc):
            N, D, R, E, _, A, _, on = _trace(sc, *_pixel_rays(c, px[q]), p)
            hit = on.any(1)
            unit = torch.where(hit, N / N.norm(dim=0).clamp(min=1e-300), 0.0)
            rows.append(torch.cat([unit, torch.where(hit, D / A.clamp(min=1e-300), 0.0)[None], R, E[None]]).T)
        images.append(torch.cat(rows))
        dirs.append(_pixel_rays(c, px)[1].T.reshape(H_, W_, 3))
    images = torch.stack(images).reshape(len(cams), H_, W_, 8)
    eye = torch.stack([_camera(c)[0] for c in cams])[:, None, None]
    hit = (images[..., :3] != 0).any(-1)
    X = eye + images[..., 3:4] * torch.stack(dirs)
    nd = torch.linalg.cross(X[:, 1:-1, 2:] - X[:, 1:-1, :-2], X[:, 2:, 1:-1] - X[:, :-2, 1:-1], dim=-1)
    nd = nd / nd.norm(dim=-1, keepdim=True)
    nd = torch.where((nd * torch.stack(dirs)[:, 1:-1, 1:-1]).sum(-1, True) > 0, -nd, nd)
    ok = hit[:, 1:-1, 1:-1] & hit[:, 1:-1, 2:] & hit[:, 1:-1, :-2] & hit[:, 2:, 1:-1] & hit[:, :-2, 1:-1]
    nm = s["normal"].double()
    loss = (_pq(images[..., 4:7]) - _pq(s["target"].double())).abs().mean()
    loss = loss + (1 - (images[..., :3] * nm).sum(-1))[hit].mean()
    loss = loss + (1 - (nd * nm[:, 1:-1, 1:-1]).sum(-1))[ok].mean()
    loss = loss + (images[..., 7] - s["mask"].double()).abs().mean()
    return images, loss, {k: None for k in ("pos", "rot", "scale", "opacity", "radiance", "emissive")}


def _exact_bake(sc, s):
    p, cams = s["params"], s["cams"]
    px = torch.arange(cams[0].width * cams[0].height, device=DEV)
    total, g = s["target"].numel(), torch.zeros_like(sc["radiance"])
    loss = 0.0
    sc["radiance"].requires_grad_()
    for ci, c in enumerate(cams):
        for q in _parts(px.numel(), sc):
            R = _trace(sc, *_pixel_rays(c, px[q]), p)[2].T
            t = s["target"][ci].reshape(-1, 3)[px[q]].double()
            x = R.detach()
            d = _pq(x) - _pq(t)
            loss += float(d.abs().sum()) / total
            g += torch.autograd.grad((R * (d.sign() * _pq_slope(x) / total)).sum(), sc["radiance"])[0]
    b1, b2 = (float(torch.tensor(b)) for b in (0.9, 0.999))
    m, v = (1 - b1) * g, (1 - b2) * g * g
    step = 0.05 * (m / (1 - b1)) / ((v / (1 - b2)).sqrt() + 1e-15)
    return torch.tensor(loss, dtype=torch.float64), (sc["radiance"].detach() - step).clamp(min=0), m, v


def _exact_pt(sc, s):
    p, cam = s["params"], s["cams"][0]
    hw = cam.width * cam.height
    out = torch.zeros(hw, 3, device=DEV, dtype=torch.float64)
    for k in range(p.spp):
        for q in _parts(hw, sc):
            pix = torch.arange(hw, device=DEV)[q]
            off = _philox(pix, k, 0xFFFFFFFF, p.camera_id, p.seed)[:2] if p.flags & JITTER else (0.5, 0.5)
            O, W = _pixel_rays(cam, pix, *off)
            beta = torch.ones(3, pix.numel(), device=DEV, dtype=torch.float64)
            for depth in range(p.max_depth + 1):
                N, D, R, E, P, A, _, on = _trace(sc, O, W, p)
                emit = on.any(1) & (E > _tau(p))
                out.index_add_(0, pix[emit], (beta * R)[:, emit].T)
                j = on.any(1) & ~emit
                u = _philox(pix[j], k, depth, p.camera_id, p.seed)
                beta, N, W, O = (beta * P)[:, j], N[:, j], W[:, j], (O + D / A.clamp(min=1e-300) * W)[:, j]
                W, pix = _bounce(N / N.norm(dim=0), u[0], u[1]), pix[j]
                if p.rr_start > 0 and depth + 1 >= p.rr_start:
                    keep = beta.amax(0).clamp(max=0.95)
                    live = u[2] < keep
                    beta, O, W, pix = (beta / keep)[:, live], O[:, live], W[:, live], pix[live]
                if pix.numel() == 0:
                    break
    return (out / p.spp).reshape(cam.height, cam.width, 3)


def exact(case, seed):
    # emitter sampling: its estimator takes the library's own table order, which plain torch has no part in;
    # and what brute force cannot do in 20 seconds
    if case["kind"] == "mis" or _segments(case) * case["n"] > 1.2e11:
        return None
    s = _inputs(case, seed)
    sc = {k: v.double() for k, v in s["arrays"].items()}
    p = s["params"]
    if case["kind"] == "sb":
        return _exact_sb(sc, s)
    if case["kind"] == "bake":
        return _exact_bake(sc, s)
    with torch.no_grad():
        if case["kind"] in ("trace", "build"):
            return _exact_probe(sc, s["rays"], p, s["hits"])
        if case["kind"] == "stage0":
            return _exact_stage0(sc, s)
        if case["kind"] == "pt":
            return _exact_pt(sc, s)
        lo, hi, r, pivot, t = s["edit"]
        f32 = dict(device=DEV, dtype=torch.float32)
        low, high = torch.tensor(lo, **f32)[:, None], torch.tensor(hi, **f32)[:, None]
        inside = ((s["arrays"]["pos"] >= low) & (s["arrays"]["pos"] <= high)).all(0)
        r, pivot, t = (torch.tensor(x, **f32).double()[:, None] for x in (r, pivot, t))
        r = r / r.norm()
        a, b = r, sc["rot"]
        d = sc["pos"] - pivot
        c = 2 * _cross(a[1:].expand_as(d), d)
        moved = d + a[0] * c + _cross(a[1:].expand_as(d), c) + pivot + t
        turned = torch.cat([(a[0] * b[0] - (a[1:] * b[1:]).sum(0))[None],
                            a[0] * b[1:] + b[0] * a[1:] + _cross(a[1:].expand_as(d), b[1:])])
        sc["pos"] = torch.where(inside, moved, sc["pos"])
        sc["rot"] = torch.where(inside, turned, sc["rot"])
        seen = {k: v.float().double() for k, v in sc.items()}
        return sc["pos"], sc["rot"], _exact_zero_bounce(seen, s["cams"], p)
