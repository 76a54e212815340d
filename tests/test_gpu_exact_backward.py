"""The backward with the exact inverse Jacobian in its three forms (all corners of a cell at once, in two halves, only those that can have
a weight), roots from the solve's records and from arrays.  tests/test_host_path.py checks without a GPU which form a case runs."""
import numpy as np
import pytest

import gpu_util as gu
import oracle
from paper_2211_15601_amd import binding, workloads as wl

SMALL, LARGE = (20, 18, 9), (48, 47, 40)          # 0.2 and 4.3 MB: held by an XCD's L2, and not

# (grid, candidates, poses, points, form)
CASES = [(SMALL, True, 1, 1501, 1), (SMALL, True, 3, 257, 1), (LARGE, True, 1, 1501, 2), (LARGE, True, 2, 259, 2),
         (SMALL, False, 1, 1501, 3), (LARGE, False, 2, 259, 3)]


@pytest.mark.gpu
@pytest.mark.parametrize("dims,voxel,P,n,form", CASES, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_gradients_with_the_exact_inverse_jacobian(gpu_lib, dims, voxel, P, n, form):
    s = wl.random_affine_scene(91, dims=dims, n_bones=8, n_poses=P, n_points=n)
    x = (s["x"] * 1.2).astype(np.float32)             # roots inside the box and beyond its faces
    x[:, 3::7] = s["x"][:, :1]                        # and many at one place
    w = wl.Workload("exact", s["dims"], 8, P, s["lo"], s["hi"], s["W"], s["B"], x, s["pose"], x, 1e-5, 10.0, 30,
                    wl.INIT_VOXEL if voxel else wl.INIT_BONE, 3 if voxel else 8, (6, 5, 4, 3))
    run = gu.GpuRun(w, grad_mode=binding.FS_GRAD_EXACT_J)
    T = run.precompute()
    xc, cv, _, _ = run.solve(fused=True, slots=True)
    assert 0.1 < cv.mean()
    gxc = w.upstream_grads()
    # (strict fp32, as the kernels: where the Jacobian is nearly singular its inverse takes up what the roundings of the entries differ by)
    want = oracle.grad(w.dims, w.lo, w.hi, T, w.W, w.B, xc, None, cv, gxc, pose=w.pose if P > 1 else None, mode=1, prec="f32")
    got = [run.grad(xc, None, cv, gxc, slot=run.slot), run.grad(xc, None, cv, gxc)]
    for g in got:
        for name, a, b in zip(("gW", "gB", "gxq"), g, want):
            gu.assert_grad_close(name, a, b, f"exact {dims} {'candidates' if voxel else 'bones'} P={P} N={n}")
    np.testing.assert_array_equal(got[0][2].view(np.uint32), got[1][2].view(np.uint32))        # dL/dx': no order to differ in
    run.ctx.close()
