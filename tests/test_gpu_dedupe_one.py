"""fs_dedupe in one launch (few lanes and few points, or more than 32 lanes): sizes around its blocks and its limits, the same context again and
again (its last block clears what its blocks waited for), a packed list that is full, and the same out of a recorded graph."""
import numpy as np
import pytest
import torch

import gpu_util as gu
import oracle
from paper_2211_15601_amd import binding

pytestmark = pytest.mark.gpu


def roots_of(N, K, seed):
    rng = np.random.default_rng(seed)
    places = rng.uniform(-1, 1, (5, 3)).astype(np.float32)                   # lanes of a point share five places: duplicates, and distinct roots
    xc = places[rng.integers(0, 5, (K, N))].transpose(0, 2, 1) + rng.uniform(-4e-4, 4e-4, (K, 3, N)).astype(np.float32)
    cv = (rng.random((K, N)) < 0.6).astype(np.uint8)
    cv[:, ::5] = 0
    return np.ascontiguousarray(xc, dtype=np.float32), cv


def expected(xc, cv, cap):
    keep, count = oracle.dedupe(xc, cv, 1e-3, prec="f32")
    offs = np.concatenate([[0], np.cumsum(count)]).astype(np.int32)
    n, k = np.nonzero(keep.T)
    return keep, offs, xc[k, :, n][:cap], k.astype(np.int32)[:cap]


def check(out, ref, cap):
    keep, offs, roots, lane = (t.cpu().numpy() for t in out)
    np.testing.assert_array_equal(keep, ref[0])
    np.testing.assert_array_equal(offs, ref[1])
    m = len(ref[3])
    np.testing.assert_array_equal(roots[:m].view(np.uint32), ref[2].view(np.uint32))
    np.testing.assert_array_equal(lane[:m], ref[3])
    assert (lane[m:] == -9).all() and np.isnan(roots[m:]).all()


@pytest.mark.parametrize("K,N", [(1, 1), (3, 37), (3, 1023), (4, 1024), (4, 1025), (3, 16384), (3, 16385), (33, 1), (33, 127), (40, 128), (64, 129), (52, 3001),
                                 (33, 128 * 1024), (33, 128 * 1024 + 1)])
def test_one_launch(gpu_lib, K, N):
    ctx = binding.Context((4, 4, 4), 2, (-1, -1, -1), (1, 1, 1))
    xc, cv = roots_of(N, K, K * 7 + N)
    d_xc, d_cv = gu.dev(xc), gu.dev(cv)
    total = int(oracle.dedupe(xc, cv, 1e-3, prec="f32")[1].sum())

    def call(cap):
        out = (torch.full((K, N), 9, dtype=torch.uint8, device=gu.DEV), torch.full((N + 1,), -9, dtype=torch.int32, device=gu.DEV),
               torch.full((K * N, 3), float("nan"), device=gu.DEV), torch.full((K * N,), -9, dtype=torch.int32, device=gu.DEV))
        ctx.dedupe(d_xc, d_cv, N, K, 1e-3, *out, cap)
        torch.cuda.synchronize()
        return out

    for cap in (K * N, total // 2, 0, K * N):
        check(call(cap), expected(xc, cv, cap), cap)


def test_one_launch_from_a_graph(gpu_lib):
    stream = torch.cuda.Stream()
    with torch.cuda.stream(stream):
        ctx = binding.Context((4, 4, 4), 2, (-1, -1, -1), (1, 1, 1), stream=stream.cuda_stream)
        K, N = 3, 9001
        xc, cv = roots_of(N, K, 5)
        d_xc, d_cv = gu.dev(xc), gu.dev(cv)
        out = (torch.empty((K, N), dtype=torch.uint8, device=gu.DEV), torch.empty((N + 1,), dtype=torch.int32, device=gu.DEV),
               torch.empty((K * N, 3), device=gu.DEV), torch.empty((K * N,), dtype=torch.int32, device=gu.DEV))
        call = lambda: ctx.dedupe(d_xc, d_cv, N, K, 1e-3, *out, K * N)
        call()
        stream.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=stream):
            call()
        for seed in (6, 7, 8):
            xc, cv = roots_of(N, K, seed)
            d_xc.copy_(gu.dev(xc)), d_cv.copy_(gu.dev(cv))
            out[2].fill_(float("nan")), out[3].fill_(-9)
            graph.replay()
            stream.synchronize()
            check(out, expected(xc, cv, K * N), K * N)
            out[2].fill_(float("nan")), out[3].fill_(-9)
            call()                                      # eager calls between the replays use the same words
            stream.synchronize()
            check(out, expected(xc, cv, K * N), K * N)
