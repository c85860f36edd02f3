"""A group's share of LDS holds 24 stack entries per lane. Where a ray reaches
every child of a wide and deep tree, a group of four lanes needs more: it gives
the round up, and its first lane traverses alone. A tree that does this: 2^20
deleted surfels (opacity 0) in one place, which pair up into a balanced tree of
ten levels. A ray through their box reaches every node and hits none of them;
a wall stands behind. (A ray takes a few seconds: few go that way.)

Without a cut, a lane alone visits each node that its ray reaches once. A group
that gave up has visited more: that is how the tests know that it did."""
import numpy as np
import pytest
import torch

import scenegen as sg
from tests._util import gpu_scene

pytestmark = pytest.mark.gpu

N = 1 << 20


@pytest.fixture(scope="module")
def scene():
    from paper_2601_23065_amd.api import BVH
    f32 = lambda a: np.ascontiguousarray(a, dtype=np.float32)   # noqa: E731
    rng = np.random.default_rng(1)
    pos, rot = np.zeros((3, N)), np.zeros((4, N))
    rot[0] = 1.0
    scale, opacity = np.full((2, N), 0.1), np.zeros(N)
    pos[:, -1], rot[:, -1], scale[:, -1], opacity[-1] = (0, 0, 1), (1, 0, 0, 0), 2.0, 0.9
    gs = gpu_scene(sg.Scene(f32(pos), f32(rot), f32(scale), f32(opacity), f32(rng.uniform(0.1, 0.8, (3, N))),
                            f32(rng.uniform(1, 9, (3, N))), f32(np.ones(N)),
                            bounds=(np.full(3, -1.0), np.full(3, 2.0))))
    return gs, BVH(gs)


def _rays(m):
    """Every 3001st ray through the deleted surfels, the others past them (half of those on the wall)."""
    g = torch.Generator(device="cuda").manual_seed(4)
    O = torch.zeros(3, m, device="cuda")
    O[0] = torch.where(torch.arange(m, device="cuda") % 2 == 0, 2.0, 50.0)
    O[:2, ::3001] = 0.04 * torch.rand(2, O[:, ::3001].shape[1], generator=g, device="cuda") - 0.02
    O[2] = -2.0
    D = torch.zeros(3, m, device="cuda")
    D[2] = 1.0
    return O, D


def test_rays_of_groups_that_give_up(scene):
    from paper_2601_23065_amd.api import Params, trace_rays
    gs, bvh = scene
    m, full = 18_000, 140_000     # nine rays a wave: four lanes each; one lane each
    O, D = _rays(m)
    Of, Df = _rays(full)
    Of[:, :m] = O
    s1, sg_ = (torch.zeros(k, 3, dtype=torch.int32, device="cuda") for k in (full, m))
    a = trace_rays(bvh, gs, Params(), Of, Df, max_hits=4, stats=s1)
    print("lanes: visits", s1[0, 2].item(), flush=True)
    b = trace_rays(bvh, gs, Params(), O, D, max_hits=4, stats=sg_)
    print("groups: visits", sg_[0, 2].item(), flush=True)
    col = torch.arange(0, m, 3001, device="cuda")
    rest = torch.ones(m, dtype=torch.bool, device="cuda")
    rest[col] = False
    assert (s1[col, 2] > N // 4).all()
    assert (sg_[col, 2] > s1[col, 2]).all()                # the groups gave up
    assert torch.equal(sg_[rest], s1[:m][rest])            # the others did not
    for x, y in zip(b, (a[0][:, :m], a[1][:m], a[2][:m])):
        assert torch.equal(x, y)
    assert (b[2][col] == 1).all() and (b[1][col, 0] == N - 1).all()


def test_paths_of_groups_that_give_up(scene):
    from paper_2601_23065_amd import api
    gs, bvh = scene
    cam = sg.Camera((0.0, 0.0, -30.0), (0.0, 0.0, 0.0), (0.0, 1.0, 0.0), 90.0, 320, 296)
    p = api.Params(spp=2, max_depth=0, rr_start=0, seed=3)
    cg, cl = (torch.zeros(6, dtype=torch.int64, device="cuda") for _ in range(2))
    # 94,720 paths a launch: 16 items a wave, four lanes each; 189,440: one lane each
    acc = api.path_trace(bvh, gs, cam, p, 0, 1, counters=cg)
    acc = api.path_trace(bvh, gs, cam, p, 1, 1, accum=acc, counters=cg)
    print("groups: visits", cg[5].item(), flush=True)
    one = api.path_trace(bvh, gs, cam, p, 0, 2, counters=cl)
    print("lanes: visits", cl[5].item(), flush=True)
    assert torch.equal(one, acc) and int(one.max()) > 0
    assert cl[4] == cg[4] and cl[5] > 2 * (N // 4)
    assert cg[5] > cl[5]
