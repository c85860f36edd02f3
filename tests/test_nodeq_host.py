"""The 64-byte nodes of the traversal on the CPU: the library's own code that
quantises a node's boxes (write_nodeq) and tests a ray against them
(node_test), compiled for the host. A ray through a leaf's surfel has to reach
the leaf however far the node's other children lie."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from paper_2601_23065_amd import build

SHIM = r"""
#include <hip/hip_runtime.h>
#include "eag_device.h"
using namespace eag;
// Which leaves of case i's node the ray of case i reaches: out [n][4].
extern "C" void leaves_reached(int n, const float* lo, const float* hi, const int* ref, const double* O,
                               const double* W, unsigned char* out) {
  for (int i = 0; i < n; ++i) {
    float l[4][3], h[4][3];
    int r[4];
    for (int k = 0; k < 4; ++k) {
      r[k] = ref[4 * i + k];
      for (int a = 0; a < 3; ++a) {
        l[k][a] = lo[(4 * i + k) * 3 + a];
        h[k][a] = hi[(4 * i + k) * 3 + a];
      }
    }
    NodeQ node;
    write_nodeq(&node, l, h, r);
    TraceCtx tc{};
    tc.nodes = &node;
    SegStats<true, false, false> s;
    seg_begin(s, d3(O[3 * i], O[3 * i + 1], O[3 * i + 2]), d3(W[3 * i], W[3 * i + 1], W[3 * i + 2]));
    const NodeKids kd = node_test(tc, s, 0, 1e-3f * 0.99999f - 1e-6f, __builtin_inff());
    for (int k = 0; k < 4; ++k) out[4 * i + k] = kd.leaf[k] ? 1 : 0;
  }
}
"""
EMPTY = 0x7fffffff
PAD = 2e-5   # of a leaf box around its surfel, times 1 + |centre|


@pytest.fixture(scope="module")
def reached(tmp_path_factory):
    d = tmp_path_factory.mktemp("nodeq")
    src, lib = os.path.join(d, "shim.hip"), os.path.join(d, "shim.so")
    with open(src, "w") as f:
        f.write(SHIM)
    subprocess.run([build.HIPCC, *build.CFLAGS, "--offload-host-only", "-shared", src, "-o", lib], check=True,
                   capture_output=True)
    fn = ctypes.CDLL(lib).leaves_reached

    def call(lo, hi, ref, O, W):
        n = len(O)
        a = [np.ascontiguousarray(lo, np.float32), np.ascontiguousarray(hi, np.float32),
             np.ascontiguousarray(ref, np.int32), np.ascontiguousarray(O, np.float64),
             np.ascontiguousarray(W, np.float64), np.zeros((n, 4), np.uint8)]
        fn(ctypes.c_int(n), *(x.ctypes.data_as(ctypes.c_void_p) for x in a))
        return a[-1].astype(bool)
    return call


def _edge_rays(rng, n, far, on_step, axis_parallel=False, reach=5.0):
    """n nodes of a flat leaf (normal z) near the origin and a sibling `far`
    away towards -x, and for each a ray through the outermost point in x of
    the leaf's surfel: its box's upper x edge less the pad. on_step: the edge
    is the last of the 255 steps from the sibling's lower x edge."""
    step = 2.0 ** np.ceil(np.log2(far / 255.0))
    grid = float(np.spacing(np.float32(256 * step)))
    edge = np.round(rng.uniform(0.05, 1.0, n) / grid) * grid if on_step else rng.uniform(0.05, 1.0, n)
    edge = edge.astype(np.float32).astype(np.float64)
    low = edge - 255 * step if on_step else np.full(n, -far)
    lo, hi = np.zeros((n, 4, 3)), np.zeros((n, 4, 3))
    p = np.stack([edge - rng.uniform(0.02, 0.05, n), rng.uniform(-0.5, 0.5, n), rng.uniform(-0.5, 0.5, n)], 1)
    pad = PAD * (1 + np.abs(p).max(1))
    lo[:, 0], hi[:, 0] = p - 0.1, p + 0.1
    hi[:, 0, 0] = edge
    lo[:, 0, 2], hi[:, 0, 2] = p[:, 2] - pad, p[:, 2] + pad
    lo[:, 1], hi[:, 1] = p - 0.1, p + 0.1
    lo[:, 1, 0], hi[:, 1, 0] = low, low + 0.1
    ref = np.tile(np.array([~0, ~1, EMPTY, EMPTY]), (n, 1))
    X = np.stack([edge - pad, p[:, 1] + rng.uniform(-0.05, 0.05, n), p[:, 2]], 1)
    W = rng.standard_normal((n, 3))
    if axis_parallel:
        W[:, 0] = 0.0
    W[:, 2] += np.copysign(0.2, W[:, 2])
    W /= np.linalg.norm(W, axis=1)[:, None]
    O = X - rng.uniform(0.1, reach, n)[:, None] * W
    return lo, hi, ref, O, W


@pytest.mark.parametrize("on_step", [False, True])
@pytest.mark.parametrize("axis_parallel", [False, True])
@pytest.mark.parametrize("far", [1.0, 30.0, 1e3, 1e4, 1e5, 1e6])
def test_far_sibling_hides_no_edge(reached, far, on_step, axis_parallel):
    rng = np.random.default_rng(int(far) + on_step + 2 * axis_parallel)
    got = reached(*_edge_rays(rng, 4000, far, on_step, axis_parallel))
    print(f"far={far:g} on_step={on_step} axis_parallel={axis_parallel} lost={int((~got[:, 0]).sum())}")
    assert got[:, 0].all()
    assert not got[:, 2:].any()


def test_boxes_stay_tight(reached):
    """A quantised box reaches at most two steps beyond its own on either
    side: rays that pass it by three are not let through."""
    rng = np.random.default_rng(5)
    lo, hi, ref, O, W = _edge_rays(rng, 4000, 30.0, False, True)
    step = 2.0 ** np.ceil(np.log2(31.0 / 255.0))
    O[:, 0] = hi[:, 0, 0] + 3 * step
    hi[:, 1, 0] = lo[:, 1, 0] + 0.1
    lo[:, 2], hi[:, 2] = lo[:, 0] + 6 * step, hi[:, 0] + 6 * step    # keeps the node's upper corner away
    ref[:, 2] = ~2
    assert not reached(lo, hi, ref, O, W)[:, 0].any()
