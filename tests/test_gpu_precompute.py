"""fs_precompute on few blocks of nodes (bones from LDS, weights eight at a time) and just beyond: transforms with the bits of the strict-fp32
oracle for numbers of bones that fill no group of four or eight, inverses of the bones through the initial states, gradients of the bones
from few and many partial sums."""
import numpy as np
import pytest

import gpu_util as gu
import oracle
from paper_2211_15601_amd import workloads as wl

pytestmark = pytest.mark.gpu

EDGE = (57, 48, 16)          # 171 blocks of 256 nodes: two poses are 342, three 513 of at most 512


@pytest.mark.parametrize("dims,nb,P", [((3, 3, 2), 1, 1), ((5, 4, 3), 3, 2), ((8, 8, 4), 8, 1), ((9, 7, 5), 9, 1), ((20, 18, 9), 17, 3), ((16, 16, 4), 24, 1),
                                       ((12, 10, 6), 33, 1), ((12, 10, 6), 64, 8), (EDGE, 24, 2), (EDGE, 5, 3)], ids=str)
def test_transforms_inverses_and_sums(gpu_lib, dims, nb, P):
    n = 257
    s = wl.random_affine_scene(600 + nb, dims=dims, n_bones=nb, n_poses=P, n_points=n)
    w = wl.Workload("pre", s["dims"], nb, P, s["lo"], s["hi"], s["W"], s["B"], s["x"], s["pose"], s["x"], 1e-5, 10.0, 20, wl.INIT_BONE, nb, (6, 5, 4, 3))
    run = gu.GpuRun(w)
    T = run.precompute()
    np.testing.assert_array_equal(T.view(np.uint32), oracle.precompute(w.dims, w.W, w.B, prec="f32").view(np.uint32))
    ref = gu.oracle_inits(w, T)
    for a, b in zip(run.init(), ref):
        np.testing.assert_array_equal(a.view(np.uint8), b.view(np.uint8))
    out = run.solve(fused=True)
    gxc = np.random.default_rng(nb).standard_normal(out[0].shape).astype(np.float32)
    want = oracle.grad(w.dims, w.lo, w.hi, T, w.W, w.B, out[0], out[2], out[1], gxc, pose=w.pose if P > 1 else None, mode=0, prec="f64")
    for name, a, b in zip(("gW", "gB", "gxq"), run.grad(out[0], out[2], out[1], gxc), want):
        gu.assert_grad_close(name, a, b, f"{dims} {nb}")
