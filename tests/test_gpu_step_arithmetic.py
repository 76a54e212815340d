"""What a Broyden step computes in another way than it is written: the reciprocal of the update's denominator, and the cell of a
point by a median.  Same bits as the strict-fp32 oracle where these can differ: denominators that are no normal numbers, points
on and beyond the box's faces."""
import numpy as np
import pytest

import gpu_util as gu
from paper_2211_15601_amd import binding, workloads as wl

pytestmark = pytest.mark.gpu

ONCE = 768 * 256         # largest batch (pairs) that the kernels without queues take
LDS, CACHED = (12, 10, 6), (20, 18, 9)


def test_reciprocal_has_the_bits_of_the_division_for_every_float(gpu_lib):
    assert binding.microbench(binding.MB_RECIP) == 0.0


def same_bits(w, run, T, max_iters):
    with np.errstate(all="ignore"):
        x0, J0, v0 = gu.oracle_inits(w, T)
        ref = gu.oracle_solve(w, T, x0, J0, v0, max_iters=max_iters)
    for out in (run.solve(fused=True), run.solve(x0, J0, v0), run.solve(fused=True, slots=True)):
        for name, a, b in zip(("roots", "masks", "J", "iterations"), out, ref):
            num = ~np.isnan(b) if b.dtype == np.float32 else np.ones(b.shape, bool)
            np.testing.assert_array_equal(np.isnan(a) if b.dtype == np.float32 else ~num, ~num)
            a, b = (v.view(np.uint32) if v.dtype == np.float32 else v for v in (a, b))
            np.testing.assert_array_equal(a[num], b[num], err_msg=name)
    return ref


@pytest.mark.parametrize("dims", [LDS, CACHED], ids=lambda d: "x".join(map(str, d)))
@pytest.mark.parametrize("n", [37, 5003, ONCE // 8 + 5])
def test_denominators_beyond_the_normal_numbers(gpu_lib, dims, n):
    # lengths scaled by 2^-56: the denominator, a product of two lengths, starts near 2^-116 and leaves the normal numbers as the
    # steps shrink; their reciprocal then overflows.  The squared tolerance is 0: every pair ends there or at the last step
    s = wl.random_affine_scene(61, dims=dims, n_bones=8, n_points=n)
    c = np.float32(2.0 ** -56)
    B = s["B"].copy()
    B.reshape(-1, 3, 4)[:, :, 3] *= c
    w = wl.Workload("tiny", s["dims"], 8, 1, s["lo"] * c, s["hi"] * c, s["W"], B, s["x"] * c, s["pose"], s["x"] * c, 1e-23, 10.0, 20,
                    wl.INIT_BONE, 8, (6, 5, 4, 3))
    run = gu.GpuRun(w)
    ref = same_bits(w, run, run.precompute(), 20)
    assert ref[1].sum() == 0 and ref[3].min() >= 2 and ref[3].max() <= 20
    run.ctx.close()


@pytest.mark.parametrize("nb,n", [(1, ONCE + 3), (5, ONCE // 5 + 2), (17, ONCE // 17 + 9), (24, ONCE // 24 + 7)])
def test_points_on_the_faces_and_tiles_of_pairs_that_end_short(gpu_lib, nb, n):
    # pairs are handed out in tiles of eight points; the last tile here has 3, 3, 6 and 7
    s = wl.random_affine_scene(70 + nb, dims=CACHED, n_bones=nb, n_points=n, max_deg=0.0)
    x = s["x"].copy()
    B = s["B"].copy()
    B.reshape(-1, 3, 4)[:, :, 3] = 0.0                  # the bones are the identity: states and roots are the points themselves
    for a in range(3):
        x[a, a::7] = s["lo"][a]
        x[a, a + 3::7] = s["hi"][a]
    w = wl.Workload("faces", s["dims"], nb, 1, s["lo"], s["hi"], s["W"], B, x, s["pose"], x, 1e-5, 10.0, 20, wl.INIT_BONE, nb, (6, 5, 4, 3))
    run = gu.GpuRun(w)
    ref = same_bits(w, run, run.precompute(), 20)
    assert ref[1].mean() > 0.99
    run.ctx.close()
