"""fs_dedupe on sizes around the tiles of its two kernels, and on points with more distinct roots than the kernel keeps in
registers, against the oracle's rule."""
import numpy as np
import pytest
import torch

import gpu_util as gu
import oracle
from paper_2211_15601_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(1, 1), (1, 64), (31, 33), (33, 32), (257, 4), (255, 5), (257, 8), (513, 9), (100, 24), (2048 * 32, 17), (2048 * 32 + 1, 16),
                                   (2048 * 256, 1), (2048 * 256 + 1, 3)],
                         ids=lambda s: f"n{s[0]}-k{s[1]}")
def test_tiles_and_many_distinct_roots(gpu_lib, shape):
    N, K = shape
    rng = np.random.default_rng(N + K)
    # roots on a coarse lattice: some lanes of a point coincide, most points keep more than four
    xc = (rng.integers(0, 4, size=(K, 3, N)) * 0.25 + rng.normal(0.0, 1e-5, size=(K, 3, N))).astype(np.float32)
    cv = (rng.random((K, N)) < 0.8).astype(np.uint8)
    ref, count = oracle.dedupe(xc, cv, 1e-3, prec="f32")
    ctx = gu.GpuRun(wl.make_config(1, n_points=4, dims=(4, 4, 4))).ctx
    total = int(count.sum())
    cap = max(total - 1, 1)                      # one entry too few: the last one is not written
    keep = torch.full((K, N), 9, dtype=torch.uint8, device=gu.DEV)
    offs = torch.full((N + 1,), -1, dtype=torch.int32, device=gu.DEV)
    roots = torch.full((cap + 1, 3), 7.0, dtype=torch.float32, device=gu.DEV)
    lane = torch.full((cap + 1,), -7, dtype=torch.int32, device=gu.DEV)
    ctx.dedupe(gu.dev(xc), gu.dev(cv), N, K, 1e-3, keep, offs, roots, lane, cap)
    np.testing.assert_array_equal(keep.cpu().numpy(), ref)
    np.testing.assert_array_equal(offs.cpu().numpy(), np.concatenate([[0], np.cumsum(count)]))
    n_idx, k_idx = np.nonzero(ref.T)
    np.testing.assert_array_equal(lane.cpu().numpy()[:min(cap, total)], k_idx[:cap])
    np.testing.assert_array_equal(roots.cpu().numpy()[:min(cap, total)], xc[k_idx, :, n_idx][:cap])
    assert int(lane[cap].item()) == -7 and float(roots[cap, 0].item()) == 7.0
