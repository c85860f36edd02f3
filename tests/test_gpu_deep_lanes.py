"""Rays with many more hits than a k-buffer round holds, in launches large
enough to run one lane per ray, where later rounds come from the lane's hit
list: with 100 coplanar layers out of the list, with 300 in one depth bucket
past its 256 entries, so that it overflows and the rounds traverse again. The
same rays in launches small enough for groups of lanes, which keep no list,
are the reference (they are held to the float64 definition by the deep-stack
tests of the small frames)."""
import pytest
import torch

import scenegen as sg
from tests._util import coplanar_stack, gpu_scene

pytestmark = pytest.mark.gpu

LANES_PATHS = 131_072      # more paths than this: one lane each (the grid's lanes on 256 CUs)
LANES_SEGMENTS = 262_144   # more one-segment items than this


def _camera(w, h):
    """Every ray passes the stack within the layers' ellipses."""
    return sg.Camera((0.0, 0.0, -2.0), (0.0, 0.0, 0.0), (0.0, 1.0, 0.0), 5.0, w, h)


@pytest.mark.parametrize("layers", [16, 17, 100, 255, 256, 272, 273, 300])
def test_paths_by_lanes_equal_paths_by_groups(layers):
    """The list's edges: 256 entries beside the 16 of the first round."""
    from paper_2601_23065_amd import api
    gs = gpu_scene(coplanar_stack(layers, 61 + layers))
    bvh = api.BVH(gs)
    spp = 2200
    p = api.Params(spp=spp, max_depth=0, rr_start=0, seed=3, flags=1)   # jittered: every path its own ray
    cam = _camera(8, 8)
    assert 64 * spp > LANES_PATHS
    c = torch.zeros(6, dtype=torch.int64, device="cuda")
    one = api.path_trace(bvh, gs, cam, p, 0, spp, counters=c)
    acc = None
    for s in range(0, spp, 550):
        acc = api.path_trace(bvh, gs, cam, p, s, 550, accum=acc)
    plain = api.path_trace(bvh, gs, cam, p, 0, spp)    # the kernel without statistics
    assert torch.equal(one, plain)
    # a path's float32 value, summed in steps of 2^-32: equal to a rounding of each
    assert ((one - acc).abs().double() <= 2.0 ** -23 * one.abs().double() + spp).all()
    assert int(one.min()) > 0
    seg, _, rounds, _, hits, _ = c.tolist()
    assert seg == 64 * spp
    assert hits == seg * layers
    assert rounds >= seg * -(-layers // 16)


@pytest.mark.parametrize("layers", [100, 300])
def test_adjoints_by_lanes_equal_adjoints_by_groups(layers):
    """Eight equal cameras (one lane per pixel) against one (groups): the
    images are the same, and the gradients eight times one camera's. All image
    gradients are positive, so that the radiance and emission gradients are
    sums of positive terms, each rounded to float at most once (2^-24) before
    a double sum, and the result once more: 2^-22 relative is above the three
    roundings of the comparison. The other sums cancel; their terms' rounding
    is bounded by the largest sum of magnitudes, 10^3 times their largest
    value with 34,000 pixels of either sign (2^-24 sqrt(34000) is 1.1e-5)."""
    from paper_2601_23065_amd import api
    gs = gpu_scene(coplanar_stack(layers, 61 + layers))
    bvh = api.BVH(gs)
    w, h = 200, 170
    assert 8 * w * h > LANES_SEGMENTS >= w * h
    cam, p = _camera(w, h), api.Params()
    img1, st1 = api.render_stage0(bvh, gs, [cam], p)
    img8, st8 = api.render_stage0(bvh, gs, [cam] * 8, p)
    assert torch.equal(img8, img1.expand(8, -1, -1, -1))
    g = torch.Generator(device="cuda").manual_seed(layers)
    d = 0.1 + torch.rand(1, h, w, 8, generator=g, device="cuda")
    g1 = api.stage0_backward(bvh, gs, [cam], p, d, st1)
    g8 = api.stage0_backward(bvh, gs, [cam] * 8, p, d.repeat(8, 1, 1, 1), st8)
    for k in g1:
        a, b = g8[k].double(), 8 * g1[k].double()
        if k in ("radiance", "emissive"):
            assert b.min() > 0
            assert ((a - b).abs() <= 2.0 ** -22 * b).all(), k
        else:
            assert (a - b).abs().max() <= 2.0 ** -24 * 1e3 * b.abs().max(), k
    z1, z8 = api.render_zero_bounce(bvh, gs, [cam], p), api.render_zero_bounce(bvh, gs, [cam] * 8, p)
    assert torch.equal(z8, z1.expand(8, -1, -1, -1))
    d3 = d[..., :3].contiguous()
    r1 = api.zero_bounce_backward(bvh, gs, [cam], p, d3)
    r8 = api.zero_bounce_backward(bvh, gs, [cam] * 8, p, d3.repeat(8, 1, 1, 1))
    assert ((r8.double() - 8 * r1.double()).abs() <= 2.0 ** -22 * 8 * r1.double()).all()
