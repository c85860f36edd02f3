"""Work items of a launch: a wave's first ones are its own by its index, the
others come from a counter, by groups of lanes or one lane each. Every item is
worked on once, at the sizes where the split and the kernel change (2048 waves
and 131,072 lanes on 256 CUs), in a scene of few surfels and one of many."""
import pytest
import torch

import scenegen as sg
from tests._util import gpu_scene

pytestmark = pytest.mark.gpu

SIZES = [1, 2, 2047, 2048, 2049, 4095, 4096, 4097, 8193, 24_575, 24_577, 32_768, 32_769, 49_151, 49_153, 65_537, 81_921,
         98_304, 98_305, 131_072, 131_073, 262_144, 262_145, 400_001]


@pytest.fixture(scope="module", params=[300, 20_000])
def scene(request):
    from paper_2601_23065_amd.api import BVH
    gs = gpu_scene(sg.cloud_scene(request.param, seed=3))
    return gs, BVH(gs)


@pytest.mark.parametrize("m", SIZES)
def test_every_item_once(scene, m):
    """A frame one pixel high: the paths started, and the sums of three samples
    in one launch against those of one and two. (A path's float32 value carries
    about 1e-13 of its directions from one form to the other: 1e-5 of a pixel's
    sum, in steps of 2^-32, is far above that.) A pixel's 0-bounce radiance,
    which only its item writes, against the frame in a launch of its own size."""
    from paper_2601_23065_amd import api
    gs, bvh = scene
    cam = sg.Camera((0.0, 0.0, -3.0), (0.0, 0.0, 0.0), (0.0, 1.0, 0.0), 40.0 / max(m, 40), m, 1)
    p = api.Params(spp=3, max_depth=2, rr_start=0, seed=11)
    c = torch.zeros(6, dtype=torch.int64, device="cuda")
    one = api.path_trace(bvh, gs, cam, p, 0, 3, counters=c)
    assert c[1] == 3 * m
    acc = api.path_trace(bvh, gs, cam, p, 0, 1, counters=c)
    acc = api.path_trace(bvh, gs, cam, p, 1, 2, accum=acc, counters=c)
    assert c[1] == 6 * m
    assert ((one - acc).abs().double() <= 1e-5 * one.abs().double() + 3 * 2.0 ** 32 * 1e-9).all()
    img = api.render_zero_bounce(bvh, gs, [cam], p)
    img8 = api.render_zero_bounce(bvh, gs, [cam] * 3, p)
    assert not img.isnan().any() and torch.equal(img8, img.expand(3, -1, -1, -1))
    st = api.render_stage0(bvh, gs, [cam], p)[1].view(-1, 28)
    assert bool(((st[:, 25] == 0) | (st[:, 25] == 1) | (st[:, 25] == 2)).all())
