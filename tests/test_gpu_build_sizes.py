"""Builds and refits at the sizes where the builder changes its way: one block
sorts up to 4096 surfels and the radix sort the others, the clustering's last
iterations run in one block from 1024 clusters on, and inputs whose pairs
hardly merge (coincident surfels) reach that block with more clusters than it
holds in LDS, or with so many that it halves them first."""
import numpy as np
import pytest
import torch

import scenegen as sg
from tests._util import gpu_scene
from tests.test_gpu_bvh import _check_binary, _check_wide

pytestmark = pytest.mark.gpu


def _coincident(n):
    f32 = lambda a: np.ascontiguousarray(a, dtype=np.float32)   # noqa: E731
    rng = np.random.default_rng(n)
    rot = np.zeros((4, n))
    rot[0] = 1.0
    return sg.Scene(f32(np.zeros((3, n))), f32(rot), f32(np.full((2, n), 0.2)), f32(np.full(n, 0.02)),
                    f32(rng.uniform(0.1, 0.8, (3, n))), f32(rng.uniform(1.0, 10.0, (3, n))), f32(np.ones(n)),
                    bounds=(np.full(3, -1.0), np.full(3, 1.0)))


def _levels_bound(n):
    return 64 + int(np.ceil(np.log2(n)))


@pytest.mark.parametrize("n", [2, 3, 5, 1023, 1024, 1025, 2049, 4096, 4097, 12289])
def test_build_and_refit_at_the_edges(n):
    """Tree invariants of a build and of a refit after moving every third
    surfel, and a trace through the refitted tree equal to one through a fresh
    build, bit for bit."""
    from paper_2601_23065_amd.api import BVH, Params, trace_rays
    scene = sg.cloud_scene(n, seed=n)
    gs = gpu_scene(scene)
    bvh = BVH(gs)
    assert _check_binary(scene, bvh) <= _levels_bound(n)
    _check_wide(scene, bvh)
    moved = scene.copy()
    moved.pos[1, ::3] += np.float32(0.25)
    g2 = gpu_scene(moved)
    bvh.refit(g2)
    _check_binary(moved, bvh)
    _check_wide(moved, bvh)
    O, D = (torch.from_numpy(x).cuda() for x in sg.random_rays(moved, 333, seed=5))
    a = trace_rays(bvh, g2, Params(), O, D, max_hits=32)
    b = trace_rays(BVH(g2), g2, Params(), O, D, max_hits=32)
    for x, y in zip(a, b):
        assert torch.equal(x, y)


@pytest.mark.parametrize("n", [1500, 3000, 150_000])
def test_pairs_that_hardly_merge(n):
    scene = _coincident(n)
    bvh = BVH_of(scene)
    assert _check_binary(scene, bvh) <= _levels_bound(n)
    _check_wide(scene, bvh)


def BVH_of(scene):
    from paper_2601_23065_amd.api import BVH
    return BVH(gpu_scene(scene))


@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
def test_a_surfel_that_is_nowhere_hides_no_other(bad):
    """A centre that is infinite or not a number is never hit, and its boxes
    hide nothing: the others trace as in the scene without it."""
    from paper_2601_23065_amd.api import BVH, Params, trace_rays
    scene = sg.cloud_scene(700, seed=4)
    scene.pos[0, 311] = bad
    gs = gpu_scene(scene)
    without = scene.copy()
    without.pos[0, 311] = 0.0
    without.opacity[311] = 0.0
    g2 = gpu_scene(without)
    O, D = (torch.from_numpy(x).cuda() for x in sg.random_rays(without, 333, seed=6))
    a = trace_rays(BVH(gs), gs, Params(), O, D, max_hits=64)
    b = trace_rays(BVH(g2), g2, Params(), O, D, max_hits=64)
    for x, y in zip(a, b):
        assert torch.equal(x, y)


def _half_coincident(n):
    """A cloud whose every other surfel lies in one place, the same way."""
    scene = sg.cloud_scene(n, seed=n)
    scene.pos[:, ::2] = 0.0
    scene.rot[:, ::2] = np.array([[1.0], [0.0], [0.0], [0.0]], np.float32)
    scene.scale[:, ::2] = 0.05
    return scene


@pytest.mark.parametrize("make", [_coincident, _half_coincident])
@pytest.mark.parametrize("n", [33_000, 100_000, 300_000])
def test_pairs_that_hardly_merge_are_halved_by_the_whole_chip(make, n):
    """More such clusters than the last block is left with: the wide iterations
    halve them. The tree stays valid, before and after a refit, and a build and
    a refit take at most four times as long as an ordinary scene's (left to the
    block they took 10 to 30 times as long, now 1 to 2)."""
    from paper_2601_23065_amd.api import BVH
    scene = make(n)
    gs, ordinary = gpu_scene(scene), gpu_scene(sg.cloud_scene(n, seed=1))
    bvh, other = BVH(gs), BVH(ordinary)
    assert _check_binary(scene, bvh) <= _levels_bound(n)
    _check_wide(scene, bvh)
    bvh.refit(gs)
    _check_binary(scene, bvh)
    _check_wide(scene, bvh)

    def best(f):
        times = []
        for _ in range(8):
            a, b = torch.cuda.Event(True), torch.cuda.Event(True)
            a.record()
            f()
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b))
        return min(times)
    build, build0 = best(lambda: BVH(gs)), best(lambda: BVH(ordinary))
    refit, refit0 = best(lambda: bvh.refit(gs)), best(lambda: other.refit(ordinary))
    print(f"n={n} build {build:.3f} ms against {build0:.3f}, refit {refit:.3f} against {refit0:.3f}")
    assert build <= 4 * build0
    assert refit <= 4 * refit0
