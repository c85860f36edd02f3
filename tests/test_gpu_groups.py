"""Rays carried by groups of lanes (launches with few items) against the same
rays carried by one lane each: the hits and sums of a ray do not depend on who
traverses for it: hit lists are equal, and values, which are computed in
double precision by the same expressions, agree to two units of float32 (the
compiler may fuse differently in the two forms)."""
import numpy as np
import pytest
import torch

import scenegen as sg
from tests._util import coplanar_stack, gpu_scene

pytestmark = pytest.mark.gpu

FULL = 140_000   # more rays than the grid has lanes: one lane each
ULPS = 2 * 2.0 ** -23


def _same(a, b):
    return bool(((a - b).abs() <= ULPS * b.abs() + 1e-30).all())


def _scene(which):
    if which == "cloud":
        return sg.cloud_scene(2000, seed=9)
    if which == "stack":       # 300 layers in one depth bucket: many rounds
        return coplanar_stack(300, seed=3)
    return sg.cloud_scene(1, seed=3)


@pytest.mark.parametrize("which", ["cloud", "stack", "single"])
@pytest.mark.parametrize("m", [1, 2, 255, 2048, 2049, 8191, 16_385, 40_000])
def test_trace_rays_small_batches_equal_a_full_one(which, m):
    from paper_2601_23065_amd.api import BVH, Params, trace_rays
    scene = _scene(which)
    gs = gpu_scene(scene)
    bvh = BVH(gs)
    O, D = (torch.from_numpy(x).cuda() for x in sg.random_rays(scene, 4096, seed=2))
    if which == "stack":       # through the stack, within its centres' spread
        O[2], D[:2], D[2] = -2.3, 0.0, 1.0
        O[:2] *= 0.2
    reps = -(-FULL // 4096)
    full = trace_rays(bvh, gs, Params(), O.repeat(1, reps), D.repeat(1, reps), max_hits=64)
    k = -(-m // 4096)
    small = trace_rays(bvh, gs, Params(), O.repeat(1, k)[:, :m].contiguous(), D.repeat(1, k)[:, :m].contiguous(),
                       max_hits=64)
    assert _same(small[0], full[0][:, :m])
    assert torch.equal(small[1], full[1][:m]) and torch.equal(small[2], full[2][:m])


def test_group_stack_that_does_not_fit():
    """A chain-shaped tree of 600 coincident surfels under groups of two lanes
    (48 stack entries): whichever way the group takes, the hits are those of
    one lane per ray."""
    from paper_2601_23065_amd.api import BVH, Params, trace_rays
    n, f32 = 600, lambda a: np.ascontiguousarray(a, dtype=np.float32)
    rot = np.zeros((4, n))
    rot[0] = 1.0
    scene = sg.Scene(f32(np.zeros((3, n))), f32(rot), f32(np.full((2, n), 0.2)), f32(np.full(n, 0.02)),
                     f32(np.full((3, n), 0.5)), f32(np.full((3, n), 2.0)), f32(np.ones(n)),
                     bounds=(np.full(3, -1.0), np.full(3, 1.0)))
    gs = gpu_scene(scene)
    bvh = BVH(gs)
    O = torch.zeros(3, FULL, device="cuda")
    O[0] = torch.linspace(-0.3, 0.3, FULL, device="cuda")
    O[2] = -2.3
    D = torch.zeros(3, FULL, device="cuda")
    D[2] = 1.0
    full = trace_rays(bvh, gs, Params(), O, D, max_hits=32)
    for m in (40_000, 20_000):
        part = trace_rays(bvh, gs, Params(), O[:, :m].contiguous(), D[:, :m].contiguous(), max_hits=32)
        assert _same(part[0], full[0][:, :m]) and torch.equal(part[1], full[1][:m])


@pytest.mark.parametrize("size,mis", [((64, 64), False), ((120, 104), False), ((192, 192), True)])
def test_frames_by_samples_equal_one_launch(size, mis):
    """All samples in one launch (one lane per path) and one sample a launch
    (groups) fill the same accumulator, with and without emitter sampling."""
    from paper_2601_23065_amd import api
    scene = sg.cloud_scene(2000, seed=9)
    gs = gpu_scene(scene)
    bvh = api.BVH(gs)
    cam = sg.Camera((0.0, 0.0, -3.0), (0.0, 0.0, 0.0), (0.0, 1.0, 0.0), 60.0, *size)
    spp = -(-FULL // (size[0] * size[1])) if not mis else 4
    p = api.Params(spp=spp, max_depth=4, rr_start=2, seed=11)
    em = api.Emitters(gs, p) if mis else None
    run = (lambda *a, **k: api.path_trace_mis(bvh, gs, em, cam, p, *a, **k)) if mis else \
          (lambda *a, **k: api.path_trace(bvh, gs, cam, p, *a, **k))
    one = run(0, spp)
    acc = None
    for k in range(spp):
        acc = run(k, 1, accum=acc)
    # a path's value is float32 and its directions carry about 1e-13 from one
    # form to the other: 1e-5 of a pixel's sum (2^-32 steps) is far above both
    assert ((one - acc).abs().double() <= 1e-5 * one.abs().double() + spp * 2.0 ** 32 * 1e-9).all()


@pytest.mark.parametrize("cams,size", [(1, (30, 20)), (2, (64, 64)), (8, (200, 170))])
def test_single_bounce_small_and_large_batches(cams, size):
    """The forward state and image of a camera do not depend on how many
    cameras share the call (groups against one lane per item), and neither
    does its gradient."""
    from paper_2601_23065_amd import api
    scene = sg.cloud_scene(2000, seed=9)
    gs = gpu_scene(scene)
    bvh = api.BVH(gs)
    cam = sg.Camera((0.0, 0.0, -3.0), (0.0, 0.0, 0.0), (0.0, 1.0, 0.0), 60.0, *size)
    p = api.Params(spp=4, seed=5)
    one = api.render_single_bounce(bvh, gs, [cam], p)
    many = api.render_single_bounce(bvh, gs, [cam] * cams, p)
    assert _same(one[0], many[0])
    z1, zn = api.render_zero_bounce(bvh, gs, [cam], p), api.render_zero_bounce(bvh, gs, [cam] * cams, p)
    for c in range(cams):
        assert _same(z1[0], zn[c])
    d = torch.ones(1, size[1], size[0], 3, device="cuda")
    g1 = api.zero_bounce_backward(bvh, gs, [cam], p, d)
    gn = api.zero_bounce_backward(bvh, gs, [cam] * cams, p, d.repeat(cams, 1, 1, 1))
    assert ((gn - cams * g1).abs() <= 1e-5 * cams * g1.abs() + 1e-12).all()


@pytest.mark.parametrize("w,h", [(200, 190), (31, 17)])
def test_flat_wall_rounding_does_not_depend_on_the_form(w, h):
    """On one flat wall of dark surfels the traced normal and distance do not
    depend on the opacities: their gradient is rounding alone. Groups (one
    camera) and lanes (eight cameras at the larger size) round alike: the
    forward state's doubles are equal bit for bit, and eight cameras give eight
    times one camera's gradient to float32 (the records' double sums, at most
    10^5 terms, add 1e-11 of their magnitudes)."""
    from paper_2601_23065_amd import api
    rng = np.random.default_rng(7)
    n, f32 = 500, lambda a: np.ascontiguousarray(a, dtype=np.float32)
    half = rng.uniform(0, np.pi, n)
    turn = np.array([np.sqrt(0.5), np.sqrt(0.5), 0.0, 0.0])    # +z to -y: no axis of the frame is exact
    c, s = np.cos(half), np.sin(half)
    rot = np.stack([turn[0] * c, turn[1] * c, -turn[1] * s, turn[0] * s])
    pos = np.stack([rng.uniform(-1, 1, n), np.full(n, 2.3), rng.uniform(-1, 1, n)])
    scene = sg.Scene(f32(pos), f32(rot), f32(rng.uniform(0.05, 0.1, (2, n))), f32(rng.uniform(0.6, 0.99, n)),
                     f32(np.full((3, n), 0.5)), f32(np.zeros((3, n))), f32(np.zeros(n)),
                     bounds=(np.full(3, -3.0), np.full(3, 3.0)))
    gs = gpu_scene(scene)
    bvh = api.BVH(gs)
    cam = sg.Camera((0.1, -0.4, 0.2), (0.0, 2.3, 0.0), (0.0, 0.0, 1.0), 40.0, w, h)
    p = api.Params()
    _, st1 = api.render_stage0(bvh, gs, [cam], p)
    _, st8 = api.render_stage0(bvh, gs, [cam] * 8, p)
    doubles = lambda s: s.view(-1, w * h, 28)[:, :, :24].contiguous().view(torch.int32)
    assert torch.equal(doubles(st8), doubles(st1).expand(8, -1, -1))
    d = torch.randn(1, h, w, 8, generator=torch.Generator(device="cuda").manual_seed(3), device="cuda")
    g1 = api.stage0_backward(bvh, gs, [cam], p, d, st1)
    g8 = api.stage0_backward(bvh, gs, [cam] * 8, p, d.repeat(8, 1, 1, 1), st8)
    for k in ("pos", "rot", "scale", "opacity"):
        assert (g8[k].double() - 8 * g1[k].double()).abs().max() <= 1e-6 * 8 * g1[k].abs().max()


def test_single_bounce_by_lanes_equals_groups():
    """Forward and adjoint of the single-bounce render, bounce gradients
    included: eight cameras in one call (one lane per item) against each
    camera alone with the stream id it has in the batch (groups). The forward
    state is equal bit for bit. The adjoints add a ray's gradient in another
    order (hit by hit, or by lanes and then across them), which moves doubles
    by 2^-53 of the sum of at most 10^2 terms' magnitudes and a record's float
    now and then: what is left is the final float rounding of each of the nine
    sums, and of the terms where they cancel: with N terms of either sign their
    magnitudes add up to about sqrt(N) times the sum, and N is at most 10^6."""
    from paper_2601_23065_amd import api
    scene = sg.cloud_scene(2000, seed=9)
    scene.radiance[:] = np.random.default_rng(2).uniform(0.1, 2.0, scene.radiance.shape)
    gs = gpu_scene(scene)
    bvh = api.BVH(gs)
    w, h, spp = 200, 170, 4
    assert 8 * w * h > 262_144 >= w * h * spp    # one lane per item against groups
    cams = [sg.Camera((0.3 * k - 1.0, 0.2, -3.0), (0.0, 0.0, 0.0), (0.0, 1.0, 0.0), 60.0, w, h) for k in range(8)]
    g = torch.Generator(device="cuda").manual_seed(1)
    d = torch.rand(8, h, w, 3, generator=g, device="cuda")
    rgb, state = api.render_single_bounce(bvh, gs, cams, api.Params(spp=spp, seed=5), keep_state=True)
    many = api.single_bounce_backward(bvh, gs, cams, api.Params(spp=spp, seed=5), d, state)
    total = {k: torch.zeros_like(v, dtype=torch.float64) for k, v in many.items()}
    size = {k: torch.zeros_like(v) for k, v in total.items()}
    px = w * h
    pix, r1 = state[:8 * px * 28].view(8, px * 28), state[8 * px * 28:].view(8, px * spp * 6)
    for c, cam in enumerate(cams):
        p = api.Params(spp=spp, seed=5, camera_id=c)
        rgb1, s1 = api.render_single_bounce(bvh, gs, [cam], p, keep_state=True)
        assert torch.equal(rgb1[0], rgb[c])
        assert torch.equal(s1[:px * 28].view(px, 28)[:, :26].contiguous().view(torch.int32),
                           pix[c].view(px, 28)[:, :26].contiguous().view(torch.int32))
        # (R of a sample that was not traced is not written)
        traced = pix[c].view(px, 28)[:, 25] == 2.0
        bits = lambda x: x.view(px, -1)[traced].contiguous().view(torch.int32)   # noqa: E731
        assert torch.equal(bits(s1[px * 28:]), bits(r1[c]))
        for k, v in api.single_bounce_backward(bvh, gs, [cam], p, d[c:c + 1].contiguous(), s1).items():
            total[k] += v.double()
            size[k] += v.double().abs()
    for k, v in many.items():
        assert (v.double() - total[k]).abs().max() <= 2.0 ** -24 * 1e3 * size[k].max(), k
        assert v.abs().max() > 0


@pytest.mark.parametrize("n", [300, 3000])
@pytest.mark.parametrize("m", [32_768, 32_769, 65_536, 65_537, 131_072])
def test_rays_at_the_lines_of_small_scenes(n, m):
    """With few surfels, batches run one lane per ray from smaller sizes on:
    either side of those lines, hits and values are those of a full batch."""
    from paper_2601_23065_amd.api import BVH, Params, trace_rays
    scene = sg.cloud_scene(n, seed=5)
    gs = gpu_scene(scene)
    bvh = BVH(gs)
    O, D = (torch.from_numpy(x).cuda().repeat(1, 35) for x in sg.random_rays(scene, 4096, seed=2))
    full = trace_rays(bvh, gs, Params(), O, D, max_hits=32)
    part = trace_rays(bvh, gs, Params(), O[:, :m].contiguous(), D[:, :m].contiguous(), max_hits=32)
    assert _same(part[0], full[0][:, :m])
    assert torch.equal(part[1], full[1][:m]) and torch.equal(part[2], full[2][:m])


def test_distances_at_a_bucket_edge_round_alike():
    """Rays through surfel centres exactly 2 m away, where a depth bucket
    begins: the last bit of the distance decides the bucket, and with it
    whether the surfel comes before or after its companion half a bucket
    nearer. Groups and lanes round it alike."""
    from paper_2601_23065_amd.api import BVH, Params, trace_rays
    rng = np.random.default_rng(12)
    n, f32 = 4096, lambda a: np.ascontiguousarray(a, dtype=np.float32)
    z = rng.standard_normal((3, n))
    far = f32(2.0 * z / np.linalg.norm(z, axis=0))          # 2 W, exactly
    W = far.astype(np.float64) / 2.0
    near = f32(W * (2.0 - 2.0 ** -14))
    rot = f32(rng.standard_normal((4, 2 * n)))
    scene = sg.Scene(f32(np.concatenate([far, near], 1)), rot, f32(np.full((2, 2 * n), 0.002)),
                     f32(np.full(2 * n, 0.3)), f32(np.full((3, 2 * n), 0.5)), f32(rng.uniform(1, 9, (3, 2 * n))),
                     f32(np.ones(2 * n)), bounds=(np.full(3, -2.1), np.full(3, 2.1)))
    gs = gpu_scene(scene)
    bvh = BVH(gs)
    D = torch.from_numpy(W).cuda()
    O = torch.zeros_like(D)
    full = trace_rays(bvh, gs, Params(), O.repeat(1, 35), D.repeat(1, 35), max_hits=8)
    part = trace_rays(bvh, gs, Params(), O, D, max_hits=8)
    first = full[1][:n, 0] < n
    both = full[2][:n] >= 2
    print(f"rays with both {int(both.sum())}, far surfel first {int((first & both).sum())}")
    assert both.sum() > n // 2 and (first & both).any() and (~first & both).any()   # the last bit does decide
    assert torch.equal(part[1], full[1][:n]) and torch.equal(part[0], full[0][:, :n])


@pytest.mark.parametrize("which", ["cloud", "room"])
def test_values_do_not_depend_on_the_form(which):
    """Every value of a ray, bit for bit, by groups of 64 to four lanes and by
    one lane each."""
    from paper_2601_23065_amd.api import BVH, Params, trace_rays
    scene = sg.cloud_scene(2000, seed=9) if which == "cloud" else sg.perturb(sg.room_scene(20_000, seed=2), seed=3)
    gs = gpu_scene(scene)
    bvh = BVH(gs)
    O, D = (torch.from_numpy(x).cuda().repeat(1, 35) for x in sg.random_rays(scene, 4096, seed=2))
    full = trace_rays(bvh, gs, Params(), O, D, max_hits=64)
    for m in (500, 3000, 6000, 12_000, 30_000):
        part = trace_rays(bvh, gs, Params(), O[:, :m].contiguous(), D[:, :m].contiguous(), max_hits=64)
        for a, b in zip(part, (full[0][:, :m], full[1][:m], full[2][:m])):
            assert torch.equal(a, b), m


@pytest.mark.parametrize("mis", [False, True])
@pytest.mark.parametrize("depth, rr", [(2, 0), (2, 2), (3, 2), (3, 1)])
def test_many_surfels_by_groups_where_roulette_ends_paths(depth, rr, mis):
    """2^18 surfels and 102,400 paths a launch: by groups with enough rounds of
    roulette, by lanes else; 204,800 by lanes. (A path's float32 value carries
    about 1e-13 of its directions from one form to the other: 1e-5 of a pixel's
    sum, in steps of 2^-32, is far above that.)"""
    from paper_2601_23065_amd import api
    scene = sg.room_scene(2 ** 18 + 1, seed=2)
    gs = gpu_scene(scene)
    bvh = api.BVH(gs)
    cam = sg.interior_cameras(scene, 1, 320, 320, seed=4)[0]
    p = api.Params(spp=2, max_depth=depth, rr_start=rr, seed=5)
    em = api.Emitters(gs, p) if mis else None
    c = torch.zeros(6, dtype=torch.int64, device="cuda")
    run = (lambda *a, **k: api.path_trace_mis(bvh, gs, em, cam, p, *a, counters=c, **k)) if mis else \
        (lambda *a, **k: api.path_trace(bvh, gs, cam, p, *a, counters=c, **k))
    one = run(0, 2)
    acc = run(0, 1)
    acc = run(1, 1, accum=acc)
    assert c[1] == 4 * 102_400 and one.abs().max() > 0
    assert ((one - acc).abs().double() <= 1e-5 * one.abs().double() + 2 * 2.0 ** 32 * 1e-9).all()
