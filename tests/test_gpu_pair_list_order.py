"""The list of pairs that have a candidate on both sides of the grid size up to which its parts lie in any order: solves of several lengths on one
context, and one that is recorded and replayed, have the results of the points alone."""
import numpy as np
import pytest
import torch

import gpu_util as gu
from paper_2211_15601_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims", [(48, 46, 39), (48, 47, 39)], ids=["in_l2", "beyond_l2"])      # 4,133,376 and 4,223,232 bytes; the line is at 4,194,304
def test_lists_and_replays(gpu_lib, dims):
    first = None
    for n in (150001, 100003, 150001):
        s = wl.random_affine_scene(19, dims=dims, n_bones=6, n_poses=1, n_points=150001)
        w = wl.Workload("list", s["dims"], 6, 1, s["lo"], s["hi"], s["W"], s["B"], s["x"], None, s["x"], 1e-5, 10.0, 20, wl.INIT_VOXEL, 3, (6, 5, 4, 3))
        if first is None:
            run = gu.GpuRun(w)
            T = run.precompute()
        run.xq, run.N = gu.dev(np.ascontiguousarray(w.xq[:, :n])), n
        out = run.solve(fused=True, slots=True)
        if first is None:
            first = out
            pick = np.arange(0, n, 997)
            ws = wl.Workload(**{**w.__dict__, "xq": np.ascontiguousarray(w.xq[:, pick])})
            x0, J0, v0 = gu.oracle_inits(ws, T)
            oxc, ocv, oJ, oit = gu.oracle_solve(ws, T, x0, J0, v0)
            np.testing.assert_array_equal(out[1][:, pick], ocv)
            np.testing.assert_array_equal(out[0][:, :, pick].view(np.uint32), oxc.view(np.uint32))
            assert out[1].sum() > 0
        for a, b in zip(out, first):
            np.testing.assert_array_equal(a, b[..., :n])
    K, N = 3, 150001
    st = torch.cuda.Stream()
    with torch.cuda.stream(st):
        run2 = gu.GpuRun(w)
        xc, cv, it = (torch.empty((K, 3, N), device=gu.DEV), torch.empty((K, N), dtype=torch.uint8, device=gu.DEV),
                      torch.empty((K, N), dtype=torch.uint8, device=gu.DEV))
        go = lambda: (run2.ctx.precompute(run2.W, run2.B), run2.ctx.solve(run2.xq, None, N, K, None, None, None, xc, cv, None, it))
        go()
        torch.cuda.synchronize()
        g = torch.cuda.CUDAGraph()
        with torch.cuda.graph(g, stream=st):
            go()
        for _ in range(3):
            xc.zero_()
            cv.zero_()
            g.replay()
            torch.cuda.synchronize()
            np.testing.assert_array_equal(cv.cpu().numpy(), first[1])
            np.testing.assert_array_equal(xc.cpu().numpy().view(np.uint32), first[0].view(np.uint32))
            go()                            # eager work between the replays
    torch.cuda.synchronize()
