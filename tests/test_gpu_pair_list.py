"""The list of pairs that have a candidate, made in one kernel: batches around its block sizes, and several solves of
different lengths on one context (the list's length is kept by the library between its kernels)."""
import numpy as np
import pytest

import gpu_util as gu
from paper_2211_15601_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(20, 18, 9), (12, 10, 6)], ids=["grid_cached", "grid_in_lds"])
def test_lists_of_several_lengths_on_one_context(gpu_lib, dims):
    # 2048, 4096 and 8192 points per block; ragged last blocks; the largest first, then shorter ones
    nb, P = 6, 2
    for n in ((1 << 21) + 1, (1 << 19) + 4097, (1 << 19) - 3, 100003):
        s = wl.random_affine_scene(411, dims=dims, n_bones=nb, n_poses=P, n_points=n)
        w = wl.Workload("list", s["dims"], nb, P, s["lo"], s["hi"], s["W"], s["B"], s["x"], s["pose"], s["x"], 1e-5, 10.0, 20,
                        wl.INIT_VOXEL, 3, (6, 5, 4, 3))
        if n == (1 << 21) + 1:
            run = gu.GpuRun(w)
            T = run.precompute()
        run.w, run.xq, run.pose, run.N = w, gu.dev(w.xq), gu.dev(w.pose), n
        first = run.solve(fused=True, slots=True)
        slot = run.slot.cpu().numpy()
        again = run.solve(fused=True, want_J=False)
        for a, b in ((first[0], again[0]), (first[1], again[1]), (first[3], again[3])):
            np.testing.assert_array_equal(a.view(np.uint8), b.view(np.uint8))
        # every point is independent of the others: the oracle solves a sample of them, the ends of the blocks among it
        pick = np.unique(np.concatenate([np.arange(0, n, 4099), np.arange(1020, n, 131072), [n - 2, n - 1]]))
        ws = wl.Workload(**{**w.__dict__, "xq": np.ascontiguousarray(w.xq[:, pick]), "pose": np.ascontiguousarray(w.pose[pick])})
        x0, J0, v0 = gu.oracle_inits(ws, T)
        oxc, ocv, oJ, oit = gu.oracle_solve(ws, T, x0, J0, v0)
        np.testing.assert_array_equal(first[1][:, pick], ocv)
        np.testing.assert_array_equal(first[3][:, pick], oit)
        np.testing.assert_array_equal(first[0][:, :, pick].view(np.uint32), oxc.view(np.uint32))
        np.testing.assert_array_equal(first[2][:, :, pick].view(np.uint32), oJ.view(np.uint32))
        assert ((slot >= 0) == (first[1] == 1)).all() and first[1].sum() > 0
