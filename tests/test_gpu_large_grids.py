"""States per bone on grids beyond the L2 of an XCD: every order in which pairs are handed out there, grids beyond 32 MiB (records asked
for ahead, no chunks dealt out), several poses.  Same bits as the strict-fp32 oracle.  tests/test_host_path.py checks without a
GPU that every case runs in the order it names."""
import numpy as np
import pytest

import gpu_util as gu
from paper_2211_15601_amd import workloads as wl

# (grid, poses, bones, points, order of roots only, order with positions): 1 tiles of eight points, 2 all states of a point side by side
CASES = [
    ((48, 47, 41), 1, 24, 8197, 1, 2),           # 4.4 MB, the last tile short
    ((96, 92, 40), 2, 24, 19003, 2, 2),          # 33.9 MB
    ((128, 128, 32), 1, 5, 120003, 2, 2),        # 25 MB, five states per point
    ((61, 47, 13), 4, 24, 8203, 1, 2),           # 7.2 MB in four poses
]


@pytest.mark.gpu
@pytest.mark.parametrize("dims,P,nb,n,roots_only,positions", CASES, ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_bone_states_on_large_grids(gpu_lib, dims, P, nb, n, roots_only, positions):
    s = wl.random_affine_scene(330 + nb, dims=dims, n_bones=nb, n_poses=P, n_points=n)
    w = wl.Workload("large", s["dims"], nb, P, s["lo"], s["hi"], s["W"], s["B"], s["x"], s["pose"], s["x"], 1e-5, 10.0, 15, wl.INIT_BONE, nb, (6, 5, 4, 3))
    run = gu.GpuRun(w)
    T = run.precompute()
    x0, J0, v0 = gu.oracle_inits(w, T)
    ref = gu.oracle_solve(w, T, x0, J0, v0)
    assert ref[1].mean() > 0.1          # (weights of random nodes: on a fine grid few pairs converge)
    for kw in (dict(want_J=False), dict(slots=True)):
        out = run.solve(fused=True, **kw)
        np.testing.assert_array_equal(out[1], ref[1])
        np.testing.assert_array_equal(out[3], ref[3])
        np.testing.assert_array_equal(out[0].view(np.uint32), ref[0].view(np.uint32))
    np.testing.assert_array_equal(out[2].view(np.uint32), ref[2].view(np.uint32))
    slot = run.slot.cpu().numpy()
    assert ((slot >= 0) == (ref[1] == 1)).all()
    gxc = w.upstream_grads()
    with_positions = run.grad(out[0], None, out[1], gxc, slot=run.slot)
    for point_major in (1, 0):           # on request, whatever the library would choose
        run.ctx.set_tuning(point_major=point_major)
        for a, b in zip(run.solve(fused=True), ref):
            np.testing.assert_array_equal(a.view(np.uint8), b.view(np.uint8))
    # the positions are a place for every root: the sums with and without them agree
    for name, a, b in zip(("gW", "gB", "gxq"), with_positions, run.grad(out[0], out[2], out[1], gxc)):
        gu.assert_grad_close(name, a, b, f"{dims} P={P}")
    run.ctx.close()
