"""Lists of nodes per correspondence cell, in chunks of one brick each: one cell with everything in it, from one chunk to more than its table holds and
from fewer samples than are kept in registers to more, on both sides of 512; flat and long grids, whose bricks are long along one axis.  Everything is
compared bit by bit, also when the grid is built again with another pose in between."""
import numpy as np
import pytest

import gpu_util as gu
import oracle
from paper_2211_15601_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dims,P,corr", [
    ((2, 2, 16), 1, (1, 1, 1, 3)), ((2, 2, 128), 1, (1, 1, 1, 8)), ((3, 3, 57), 1, (1, 1, 1, 8)),       # 64, 512 and 513 nodes in one chunk
    ((2, 2, 256), 1, (1, 1, 1, 3)), ((2, 2, 257), 1, (1, 1, 1, 3)),         # a whole brick, and one row more
    ((2, 2, 2048), 1, (1, 1, 1, 2)), ((2, 2, 2049), 2, (1, 1, 1, 2)),       # eight chunks, nine
    ((2, 700, 3), 1, (2, 2, 2, 3)), ((700, 2, 3), 1, (2, 2, 2, 3)),         # bricks along y, along x
    ((9, 9, 200), 1, (9, 9, 1, 3)), ((9, 10, 200), 3, (5, 9, 1, 8)),        # columns: more than eight chunks, up to and more than 512 nodes
    ((33, 33, 33), 2, (7, 7, 7, 3)),
], ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_candidates_equal_the_oracle(gpu_lib, dims, P, corr):
    s = wl.random_affine_scene(41, dims=dims, n_bones=5, n_poses=P, n_points=8 * P)
    w = wl.Workload("chunks", s["dims"], 5, P, s["lo"], s["hi"], s["W"], s["B"], s["x"], s["pose"] if P > 1 else None, s["x"],
                    1e-5, 10.0, 20, wl.INIT_VOXEL, 3, corr)
    run = gu.GpuRun(w)
    other = run.B.flip(1).contiguous()      # the bones in another order
    T = run.precompute()
    run.ctx.precompute(run.W, other)
    T = run.precompute()
    bbox, cand = run.corr()
    obox, ocand = oracle.corr_build(w.dims, w.lo, w.hi, T, corr, prec="f32")
    np.testing.assert_array_equal(bbox.view(np.uint32).ravel(), obox.view(np.uint32).ravel())
    np.testing.assert_array_equal(cand.ravel(), ocand.ravel())
    assert (cand >= 0).any()


@pytest.mark.parametrize("dims,P,corr", [
    ((2, 2, 129), 1, (1, 1, 1, 8)),                                         # 516 nodes: four behind those that are kept
    ((20, 20, 5), 2, (1, 1, 1, 8)), ((13, 11, 17), 1, (2, 2, 1, 8)),        # the limit inside a chunk that is not the first
    ((24, 24, 24), 1, (2, 1, 1, 8)),                                        # most behind it, in the table and in the list
], ids=lambda v: "x".join(map(str, v)) if isinstance(v, tuple) else str(v))
def test_cells_that_do_not_fit_the_registers(gpu_lib, dims, P, corr):
    test_candidates_equal_the_oracle(gpu_lib, dims, P, corr)
