"""The sorted record lists of the backward: cells with no record to thousands (pieces on both sides of the length from which
they are summed, and cut at every multiple of 256), walked as one list per node, and positions that are counted by the backward
itself, for numbers of lanes per point on both sides of the tile of 8."""
import numpy as np
import pytest

import gpu_util as gu
import oracle
from paper_2211_15601_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,K,P,N,spread", [
    ((3, 3, 3), 1, 1, 1, 1.0), ((4, 3, 5), 3, 1, 257, 0.2),         # one record; one crowded corner
    ((12, 11, 9), 7, 2, 300, 1.0), ((12, 11, 9), 8, 1, 301, 1.0), ((12, 11, 9), 9, 3, 299, 0.5),
    ((20, 18, 33), 2, 1, 6000, 1.0), ((20, 18, 33), 17, 2, 511, 0.3),    # columns of more than half a wave; sparse and crowded cells in one column
    ((6, 5, 70), 24, 1, 1000, 0.6),                                 # columns longer than a wave
], ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_gradient_of_given_roots(gpu_lib, dims, K, P, N, spread):
    s = wl.random_affine_scene(61, dims=dims, n_bones=4, n_poses=P, n_points=N)
    w = wl.Workload("lists", s["dims"], 4, P, s["lo"], s["hi"], s["W"], s["B"], s["x"], s["pose"] if P > 1 else None, s["x"],
                    1e-5, 10.0, 20, wl.INIT_BONE, 4, (1, 1, 1, 1))
    run = gu.GpuRun(w)
    run.K = K                       # fs_grad takes any number of lanes per point
    T = run.precompute()
    rng = np.random.default_rng(N)
    lo, hi = np.asarray(s["lo"]), np.asarray(s["hi"])
    u = rng.random((K, 3, N)) ** (1.0 / spread)                     # spread < 1: towards the lower corner of the box
    u[:, :, ::5] = u[:1, :, ::5]                                    # every fifth point: all lanes at one root
    xc = (lo[None, :, None] + u * (hi - lo)[None, :, None]).astype(np.float32)
    J = (np.eye(3).reshape(1, 9, 1) + 0.2 * rng.standard_normal((K, 9, N))).astype(np.float32)
    cv = (rng.random((K, N)) < 0.8).astype(np.uint8)
    gxc = rng.standard_normal((K, 3, N)).astype(np.float32)
    want = oracle.grad(w.dims, w.lo, w.hi, T, w.W, w.B, xc, J, cv, gxc, pose=w.pose, mode=0, prec="f64")
    got = run.grad(xc, J, cv, gxc)
    for name, a, b in zip(("gW", "gB", "gxq"), got, want):
        gu.assert_grad_close(name, a, b, f"{dims} K={K} P={P} N={N}")
