"""k_solve_ws: how the pairs reach the waves.  Every consumer prepares its first pairs itself, at most 64, the producers what is behind those,
and all waves take from one queue per block: batches around the sizes where the one ends and the other begins, lists of candidates that
leave most waves, or all of them, without a pair.  Same bits as the strict-fp32 oracle."""
import numpy as np
import pytest
import torch

import gpu_util as gu
from paper_2211_15601_amd import workloads as wl

pytestmark = pytest.mark.gpu

DIMS, NB = (20, 18, 9), 8
BLOCKS = 3 * 256                        # grid of 152 KiB: three blocks per compute unit, three consumers each
OWN = BLOCKS * 3 * 64                   # pairs of a batch that the consumers prepare themselves
CHUNK = 128                             # pairs per block below which there are fewer blocks


@pytest.mark.parametrize("pairs", [8, 8 * 16, CHUNK * BLOCKS - 8, CHUNK * BLOCKS + 8, OWN - 8, OWN, OWN + 8, OWN + CHUNK * 3 + 8, OWN + CHUNK * BLOCKS + 8])
def test_batches_around_what_the_consumers_prepare(gpu_lib, pairs):
    # solved in place (the query points lie in the roots' array), which takes this kernel whatever the size
    n = pairs // NB
    s = wl.random_affine_scene(411, dims=DIMS, n_bones=NB, n_points=n)
    w = wl.Workload("queue", s["dims"], NB, 1, s["lo"], s["hi"], s["W"], s["B"], s["x"], s["pose"], s["x"], 1e-5, 10.0, 50, wl.INIT_BONE, NB, (6, 5, 4, 3))
    run = gu.GpuRun(w)
    T = run.precompute()
    ref = gu.oracle_solve(w, T, *gu.oracle_inits(w, T))
    new = lambda *shape, dtype=torch.float32: torch.full(shape, 99, dtype=dtype, device=gu.DEV)
    for positions in (False, True):
        xc, J, cv, it, slot = new(NB, 3, n), new(NB, 9, n), new(NB, n, dtype=torch.uint8), new(NB, n, dtype=torch.uint8), new(NB, n, dtype=torch.int32)
        xc[0].copy_(run.xq)
        run.ctx.solve(xc[0], None, n, NB, None, None, None, xc, cv, J if positions else None, it, slot if positions else None)
        torch.cuda.synchronize()
        for name, a, b in (("roots", xc, ref[0]), ("masks", cv, ref[1]), ("iterations", it, ref[3])) + ((("J", J, ref[2]),) if positions else ()):
            np.testing.assert_array_equal(a.cpu().numpy().view(np.uint8), b.view(np.uint8), err_msg=f"{name} {positions}")
        if positions:
            assert ((slot.cpu().numpy() >= 0) == (ref[1] == 1)).all()


@pytest.mark.parametrize("laps", [2, 4])
def test_queue_used_several_times_over(gpu_lib, laps):
    # a round of the queue is 192 entries per block; few steps per pair, so that the producers' waves change their priority as the queue runs empty
    n = (OWN + laps * 192 * BLOCKS) // NB
    s = wl.random_affine_scene(414, dims=DIMS, n_bones=NB, n_points=n)
    w = wl.Workload("laps", s["dims"], NB, 1, s["lo"], s["hi"], s["W"], s["B"], s["x"], s["pose"], s["x"], 1e-5, 10.0, 50, wl.INIT_BONE, NB, (6, 5, 4, 3))
    run = gu.GpuRun(w)
    T = run.precompute()
    ref = gu.oracle_solve(w, T, *gu.oracle_inits(w, T))
    for kw in (dict(want_J=False), dict(slots=True)):
        out = run.solve(fused=True, **kw)
        for name, a, b in zip(("roots", "masks", "J", "iterations"), out, ref):
            if a is not None:
                np.testing.assert_array_equal(a.view(np.uint8), b.view(np.uint8), err_msg=f"{name} {sorted(kw)}")


@pytest.mark.parametrize("some", [0, 1, 700, 33000])
def test_lists_that_leave_waves_without_a_pair(gpu_lib, some):
    corr, n = (24, 24, 12, 3), 294912 // 3 + 1                      # just above the batches that need no list
    s = wl.random_affine_scene(412, dims=DIMS, n_bones=NB, n_points=n)
    w = wl.Workload("sparse", s["dims"], NB, 1, s["lo"], s["hi"], s["W"], s["B"], s["x"], s["pose"], s["x"], 1e-5, 10.0, 30, wl.INIT_VOXEL, 3, corr)
    run = gu.GpuRun(w)
    run.precompute()
    bbox, cand = run.corr()
    cell = int(np.flatnonzero(cand[0, :, 0] < 0)[0])               # a cell without candidates: all points but `some` lie there
    at = np.array([cell // (corr[1] * corr[2]), cell // corr[2] % corr[1], cell % corr[2]])
    lo, hi = bbox[0, :3], bbox[0, 3:]
    x = np.repeat((lo + (at + 0.5) * (hi - lo) / np.array(corr[:3])).astype(np.float32)[:, None], n, axis=1)
    x[:, :some] = s["x"][:, :some]
    w.xq = x
    run = gu.GpuRun(w)
    T = run.precompute()
    x0, J0, v0 = gu.oracle_inits(w, T)
    ref = gu.oracle_solve(w, T, x0, J0, v0)
    assert v0.sum() >= some * 0.1 and v0[:, some:].sum() == 0
    for kw in (dict(want_J=False), dict(slots=True)):
        out = run.solve(fused=True, **kw)
        for name, a, b in zip(("roots", "masks", "J", "iterations"), out, ref):
            if a is not None:
                np.testing.assert_array_equal(a.view(np.uint8), b.view(np.uint8), err_msg=f"{name} {sorted(kw)}")


@pytest.mark.parametrize("init,n", [(wl.INIT_VOXEL, 349525), (wl.INIT_VOXEL, 349526), (wl.INIT_BONE, 196607), (wl.INIT_BONE, 196608)])
def test_given_states_claimed_whole(gpu_lib, init, n):
    # around 2048 pairs per block (two blocks per compute unit with candidates, else three), where waves begin to claim all that they have lanes for
    # or nothing: the bits of the solve that makes the same states itself, and whose waves take what there is
    K = NB if init == wl.INIT_BONE else 3
    s = wl.random_affine_scene(413, dims=DIMS, n_bones=NB, n_points=n)
    w = wl.Workload("given", s["dims"], NB, 1, s["lo"], s["hi"], s["W"], s["B"], s["x"], s["pose"], s["x"], 1e-5, 10.0, 50, init, K, (6, 5, 4, 3))
    run = gu.GpuRun(w)
    run.precompute()
    new = lambda *shape, dtype=torch.float32: torch.full(shape, 99, dtype=dtype, device=gu.DEV)
    outs = []
    for given in (False, True):
        x0, J0, v0 = new(K, 3, n), new(K, 9, n), new(K, n, dtype=torch.uint8)
        xc, J, cv, it = new(K, 3, n), new(K, 9, n), new(K, n, dtype=torch.uint8), new(K, n, dtype=torch.uint8)
        if given:
            run.ctx.init(run.xq, None, n, x0, J0, v0)
        run.ctx.solve(run.xq, None, n, K, *((x0, J0, v0) if given else (None, None, None)), xc, cv, J, it)
        torch.cuda.synchronize()
        outs.append((xc, cv, J, it))
    for name, a, b in zip(("roots", "masks", "J", "iterations"), *outs):
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8)), name
    assert outs[0][1].float().mean() > 0.2
