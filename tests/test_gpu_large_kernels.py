"""The solve kernels with queues (grid in LDS: 4 or 12 waves per block; grid read through the caches: producer and consumers)
on batches just above the sizes that kernels without queues take, with the inputs in which they can go wrong: query points
that are no numbers, lanes marked invalid, no iterations.  Same bits as the strict-fp32 oracle.  tests/test_host_path.py
checks without a GPU that every case runs the kernel it names."""
import numpy as np
import pytest
import torch

import gpu_util as gu
from paper_2211_15601_amd import workloads as wl

BONE, VOXEL = 196608, 294912          # largest batches (pairs, 256 CUs) without a queue: states per bone or given / candidates
LDS4, LDS12, CACHED = (12, 10, 6), (13, 15, 16), (20, 18, 9)          # 34, 146 and 152 KiB

# (grid, bones, voxel, initial states computed inside the kernel, points, kernel with J~, kernel without)
CASES = [
    (LDS4, 24, False, True, BONE // 24 + 1, "k_solve<true,true,4>", "k_solve<true,false,4>"),
    (LDS4, 24, False, False, BONE // 24 + 1, "k_solve<false,true,4>", "k_solve<false,false,4>"),
    (LDS4, 6, True, True, VOXEL // 3 + 1, "k_solve<true,true,4>", "k_solve<true,false,4>"),
    (LDS12, 24, False, True, BONE // 24 + 1, "k_solve<true,true,12>", "k_solve<true,false,12>"),
    (LDS12, 24, False, False, BONE // 24 + 37, "k_solve<false,true,12>", "k_solve<false,false,12>"),
    (LDS12, 6, True, True, VOXEL // 3 + 1, "k_solve<true,true,12>", "k_solve<true,false,12>"),
    (LDS12, 6, True, False, BONE // 3 + 1, "k_solve<false,true,12>", "k_solve<false,false,12>"),
    (CACHED, 24, False, True, BONE // 24 + 1, "k_solve_ws<true,true,3,true>", "k_solve_ws<true,false,3,true>"),
    (CACHED, 24, False, False, BONE // 24 + 37, "k_solve_ws<false,true,3,true>", "k_solve_ws<false,false,3,true>"),
    (CACHED, 6, True, True, VOXEL // 3 + 1, "k_solve_ws<true,true,3,false>", "k_solve_ws<true,false,3,false>"),
    (CACHED, 6, True, False, BONE // 3 + 1, "k_solve_ws<false,true,3,false>", "k_solve_ws<false,false,3,false>"),
]


def case_id(c):
    return f"{c[5].split('<')[0]}-g{c[0][0]}x{c[0][1]}x{c[0][2]}-{'voxel' if c[2] else 'bone'}-{'fused' if c[3] else 'given'}"


@pytest.mark.gpu
@pytest.mark.parametrize("case", CASES, ids=case_id)
def test_edge_inputs_above_the_small_batch_limits(gpu_lib, case):
    dims, nb, voxel, fused, n, _, _ = case
    s = wl.random_affine_scene(500 + nb, dims=dims, n_bones=nb, n_poses=1, n_points=n)
    xq = s["x"].copy()
    xq[1, 5::4001] = np.nan
    xq[0, 7::4003] = np.inf
    xq[2, n - 1] = -np.inf
    w = wl.Workload("edge", s["dims"], nb, 1, s["lo"], s["hi"], s["W"], s["B"], xq, s["pose"], xq, 1e-5, 10.0, 50,
                    wl.INIT_VOXEL if voxel else wl.INIT_BONE, 3 if voxel else nb, (6, 5, 4, 3))
    for max_iters in (50, 0):
        run = gu.GpuRun(w, max_iters=max_iters)
        T = run.precompute()
        with np.errstate(all="ignore"):
            x0, J0, v0 = gu.oracle_inits(w, T)
            if not fused:
                v0[1, 3::1009] = 0
                v0[:, 11::2003] = 0
            ref = gu.oracle_solve(w, T, x0, J0, v0, max_iters=max_iters)
        for kw in (dict(slots=True), dict(want_J=False)):
            out = run.solve(fused=True, **kw) if fused else run.solve(x0, J0, v0, **kw)
            np.testing.assert_array_equal(out[1], ref[1])
            np.testing.assert_array_equal(out[3], ref[3])
            for name, a, b in (("roots", out[0], ref[0]), ("J", out[2], ref[2])):
                if a is None:
                    continue
                num = ~np.isnan(b)          # a NaN has no bits of its own
                assert (np.isnan(a) == ~num).all(), (name, max_iters)
                np.testing.assert_array_equal(a.view(np.uint32)[num], b.view(np.uint32)[num], err_msg=f"{name} {max_iters}")
            if kw.get("slots"):
                slot = run.slot.cpu().numpy()
                assert ((slot >= 0) == (ref[1] == 1)).all()
        if max_iters:
            assert 0 < ref[1].sum() < ref[1].size and (ref[1][:, 5] == 0).all()
        run.ctx.close()


@pytest.mark.gpu
@pytest.mark.parametrize("n", [BONE // 24 + 1, 4001])
@pytest.mark.parametrize("weight, far", [(1.5e38, 1.0), (1e15, 1e25)])
def test_products_beyond_the_largest_number(gpu_lib, n, weight, far):
    # Nodes next to two faces of the box blend to numbers whose product with a position is infinite, though the entries
    # are finite.  For a state clamped to such a face they are corners of weight zero, and 0 * inf is no number: the
    # kernels that do not fetch corners of weight zero must give what fs_init gives.
    s = wl.random_affine_scene(517, dims=CACHED, n_bones=24, n_poses=1, n_points=n)
    W = s["W"].copy()
    W[1, :, :, 3] = weight
    W[2:, -2, :, 5] = weight
    xq = (s["x"] * np.where(np.arange(n) % 3 == 0, far, 1.0)).astype(np.float32)
    w = wl.Workload("beyond", s["dims"], 24, 1, s["lo"], s["hi"], W, s["B"], xq, s["pose"], xq, 1e-5, 10.0, 50, wl.INIT_BONE, 24, (6, 5, 4, 3))
    run = gu.GpuRun(w)
    T = run.precompute()
    assert np.isfinite(T).all()
    with np.errstate(all="ignore"):
        x0, J0, v0 = gu.oracle_inits(w, T)
        ref = gu.oracle_solve(w, T, x0, J0, v0)
    assert np.isnan(J0).any() or (v0 == 0).any()
    for out in (run.solve(fused=True), run.solve(x0, J0, v0)):
        np.testing.assert_array_equal(out[1], ref[1])
        np.testing.assert_array_equal(out[3], ref[3])
        for a, b in ((out[0], ref[0]), (out[2], ref[2])):
            num = ~np.isnan(b)
            np.testing.assert_array_equal(np.isnan(a), ~num)
            np.testing.assert_array_equal(a.view(np.uint32)[num], b.view(np.uint32)[num])
    run.ctx.close()


@pytest.mark.gpu
@pytest.mark.parametrize("by_place", [0, 1, 2])
def test_a_step_with_candidates_replays_from_a_hip_graph(gpu_lib, by_place):
    # k_voxel_list, or the sort, then k_solve_ws, and the scans of the grid build and of the backward: kernels that use words
    # which another kernel of the same call clears.  Every replay must find them cleared, also with eager calls in between
    n = 100003
    w = wl.make_config(5, n_points=n, dims=(32, 32, 16), n_poses=2)
    N, K = w.N, w.K
    new = lambda *shape, dtype=torch.float32: torch.empty(shape, dtype=dtype, device=gu.DEV)
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        from paper_2211_15601_amd import binding
        ctx = binding.Context(w.dims, w.n_bones, w.lo, w.hi, n_poses=w.n_poses, tol=w.tol, div_thresh=w.div_thresh, max_iters=w.max_iters,
                              init_mode=w.init_mode, corr_dims=w.corr_dims)
        ctx.set_list_order(by_place)
        W, B, xq, pose, gxc = gu.dev(w.W), gu.dev(w.B), gu.dev(w.xq), gu.dev(w.pose), gu.dev(w.upstream_grads())
        xc, cv, it, slot = new(K, 3, N), new(K, N, dtype=torch.uint8), new(K, N, dtype=torch.uint8), new(K, N, dtype=torch.int32)
        gW, gB, gxq = new(*w.W.shape), new(*w.B.shape), new(3, N)
        keep, offs, roots, lane = new(K, N, dtype=torch.uint8), new(N + 1, dtype=torch.int32), new(K * N, 3), new(K * N, dtype=torch.int32)

        def step():
            ctx.precompute(W, B)
            ctx.solve(xq, pose, N, K, None, None, None, xc, cv, None, it, slot)
            ctx.grad(W, xc, None, cv, gxc, pose, N, K, gW, gB, gxq, slot)
            ctx.dedupe(xc, cv, N, K, 1e-3, keep, offs, roots, lane, K * N)

        roots.zero_()
        lane.zero_()
        step()                                   # eager: also sizes the library's buffers
        side.synchronize()
        exact = (xc, cv, it, keep, offs, roots, lane)
        ref, ref_grad = [t.clone() for t in exact], [t.clone() for t in (gW, gB, gxq)]
        assert cv.sum().item() > 0
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=side):
            step()
        side.synchronize()
        for rep in range(3):
            for t in exact + (gW, gB, gxq):
                t.zero_()
            side.synchronize()
            graph.replay()
            side.synchronize()
            for a, b in zip(exact, ref):
                assert torch.equal(a, b), rep
            for a, b in zip((gW, gB, gxq), ref_grad):
                assert ((a - b).norm() / b.norm()).item() < 2e-5, rep
            step()                               # eager work between the replays
        side.synchronize()
        ctx.close()
