"""fs_dedupe with four points per thread: batches from its first size on whose number is and is not a multiple of four (rows of any alignment, groups cut
short at a tile's end), one to four lanes, any byte for "converged"."""
import numpy as np
import pytest
import torch

import gpu_util as gu
import oracle
from paper_2211_15601_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,K", [((1 << 19) - 1, 3), (1 << 19, 4), ((1 << 19) + 1, 3), ((1 << 19) + 255, 2), ((1 << 20) + 3, 1), ((1 << 20) + 2, 4)])
def test_four_points_per_thread(gpu_lib, N, K):
    rng = np.random.default_rng(N + K)
    xc = (rng.integers(0, 2, size=(K, 3, N)) * 0.25 + rng.normal(0.0, 1e-5, size=(K, 3, N))).astype(np.float32)
    cv = rng.choice(np.array([0, 0, 1, 2, 255], np.uint8), size=(K, N))
    cv[:, ::7] = 0
    ref, count = oracle.dedupe(xc, (cv != 0).astype(np.uint8), 1e-3, prec="f32")
    ctx = gu.GpuRun(wl.make_config(1, n_points=4, dims=(4, 4, 4))).ctx
    total = int(count.sum())
    keep = torch.full((K * N + 16,), 9, dtype=torch.uint8, device=gu.DEV)
    offs = torch.full((N + 5,), -1, dtype=torch.int32, device=gu.DEV)
    roots = torch.full((total + 1, 3), 7.0, dtype=torch.float32, device=gu.DEV)
    lane = torch.full((total + 1,), -7, dtype=torch.int32, device=gu.DEV)
    ctx.dedupe(gu.dev(xc), gu.dev(cv), N, K, 1e-3, keep, offs, roots, lane, total)
    got = keep.cpu().numpy()
    np.testing.assert_array_equal(got[:K * N].reshape(K, N), ref)
    assert (got[K * N:] == 9).all() and (offs[N + 1:] == -1).all()
    np.testing.assert_array_equal(offs.cpu().numpy()[:N + 1], np.concatenate([[0], np.cumsum(count)]))
    n_idx, k_idx = np.nonzero(ref.T)
    np.testing.assert_array_equal(lane.cpu().numpy()[:total], k_idx)
    np.testing.assert_array_equal(roots.cpu().numpy()[:total], xc[k_idx, :, n_idx])
    assert int(lane[total].item()) == -7
