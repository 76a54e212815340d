"""Host code of the library on a stub runtime (host_path.py): what it launches and what it answers when memory runs out."""
import host_path
import test_gpu_exact_backward as exact
import test_gpu_large_grids as large_grids
import test_gpu_large_kernels as large


def test_positions_of_a_solve_whose_records_are_gone_are_refused(tmp_path):
    # A solve that needs more room for its records frees what it has first.  When the new allocation fails, the records of
    # the solve before are gone, and so are its positions: fs_grad must not launch a kernel that reads them.
    host_path.run("""
h, n, K = ctx((64, 64, 16)), 20000, 24
assert precompute(h) == OK and solve(h, n, K, slot=True) == OK and grad(h, n, K, slot=True) == OK
launched()
S.stub_fail_allocation(0)
assert solve(h, 2 * n, K, slot=True) == E_ALLOC
assert grad(h, n, K, slot=True) == E_STATE, names()
assert launched() == []
# the context goes on, and nothing is freed twice
assert solve(h, n, K, slot=True) == OK and grad(h, n, K, slot=True) == OK
L.fs_destroy(h)
assert S.stub_bad_frees() == 0 and S.stub_live_blocks() == 0
""", tmp_path)


def test_words_of_the_scans_are_cleared_where_no_graph_can_record_it(tmp_path):
    # The scans in one pass need words that are zero when they start; a block waits for what it reads there.  They are
    # made and cleared with the context.  Made on demand, and cleared by a launch on the stream of the call that
    # needed more of them, they stayed uncleared when that stream was recording a graph instead of running it.
    host_path.run("""
h, n, K = ctx((64, 64, 16), init=VOXEL), 1 << 23, 3
S.stub_fail_allocation(0)
assert precompute(h) == OK                  # asks for nothing: the grid and its candidates stay a pair
S.stub_fail_allocation(-1)
launched()
for k in range(1, 4):                       # every solve longer than any before
    assert solve(h, k * n, K) == OK
    assert [x.split("<")[0] for x in names()] == ["k_voxel_list", "k_solve_ws", "k_solve_unpack"]
L.fs_destroy(h)
assert S.stub_bad_frees() == 0 and S.stub_live_blocks() == 0
""", tmp_path)


def test_scans_after_a_failed_launch_find_their_words_cleared(tmp_path):
    # The kernel that clears the words is not the one that uses them: when a launch of a call has failed, nobody knows
    # what they hold, and the next scan would add it up or wait for it for ever.
    host_path.run("""
def failing(h, call, kernels):
    for i in range(kernels):
        S.stub_fail_launch(i)
        assert call() == E_DEVICE, i
        S.stub_fail_launch(-1)
        before = S.stub_memsets()
        launched()
        assert precompute(h) == OK and call() == OK
        assert S.stub_memsets() == before + 1, (i, names())
        before = S.stub_memsets()
        assert precompute(h) == OK and call() == OK and S.stub_memsets() == before

h, n, K = ctx((64, 64, 16), init=VOXEL), 1 << 20, 3
assert precompute(h) == OK and solve(h, n, K, slot=True) == OK and grad(h, n, K, slot=True) == OK
for call in (lambda: precompute(h), lambda: solve(h, n, K, slot=True), lambda: grad(h, n, K)):
    launched()
    assert call() == OK
    failing(h, call, len(launched()))
L.fs_destroy(h)
""", tmp_path)


def test_lists_are_ordered_on_request_from_the_size_the_header_states(tmp_path):
    # whatever number of candidates makes the batch small enough for a kernel without a list
    host_path.run("""
for ck in (1, 3, 8):
    h = ctx((64, 64, 16), init=VOXEL, ck=ck)
    assert precompute(h) == OK
    for order in (1, 2):
        assert L.fs_set_list_order(h, order) == OK
        for n, ordered in ((65535, False), (65536, True), (70001, True), (400000, True)):
            launched()
            for slot in (False, True):
                assert solve(h, n, ck, slot=slot) == OK
                assert ("k_sort_hist" in names()) == ordered, (ck, order, n, slot)
    assert L.fs_set_list_order(h, 0) == OK and solve(h, 65536, ck) == OK and "k_sort_hist" not in names()
    L.fs_destroy(h)
""", tmp_path)


def test_small_batches_copy_the_grid_into_lds_only_where_a_block_has_the_waves_for_it(tmp_path):
    # A batch of no more waves than the GPU has compute units runs in blocks of one wave: one that first copies a grid
    # of 146 KiB takes longer than the whole call does through the caches.
    host_path.run("""
def kernel(h, n, K, **kw):
    launched()
    assert solve(h, n, K, **kw) == OK
    (k,) = [x for x in launched() if x[0].startswith("k_solve_")]
    return k[0].replace(" ", ""), k[2][0] // 64, k[3]

h = ctx((13, 15, 16))
big = 13 * 15 * 16 * 48
assert precompute(h) == OK
for kw, im in ((dict(), 0), (dict(slot=True), 0), (dict(fused=False, J=True), 2)):
    for n in (1, 37, 160, 300):                      # one or two waves per block
        assert kernel(h, n, 24, **kw) == (f"k_solve_quad<{im},false>", 4, 0), n
    for n, waves in ((400, 3), (1000, 6), (2048, 12)):
        assert kernel(h, n, 24, **kw) == (f"k_solve_quad<{im},true>", waves, big), n
    assert kernel(h, 8192, 24, **kw) == (f"k_solve_once<{im},true>", 12, big)
L.fs_destroy(h)
h = ctx((16, 16, 4))                                 # 48 KiB
assert precompute(h) == OK and kernel(h, 1, 24) == ("k_solve_quad<0,true>", 1, 48 << 10)
L.fs_destroy(h)
h = ctx((16, 16, 4), init=VOXEL)
assert precompute(h) == OK
assert kernel(h, 500, 3) == ("k_solve_quad<1,false>", 4, 0) and kernel(h, 2000, 3) == ("k_solve_quad<1,true>", 2, 48 << 10)
assert L.fs_set_tuning(h, 0, 0, 0, -1, 0) == OK and kernel(h, 2000, 3) == ("k_solve_quad<1,false>", 4, 0)
L.fs_destroy(h)
h = ctx((13, 15, 17))                                # larger than what is kept in LDS
assert precompute(h) == OK and kernel(h, 8192, 24) == ("k_solve_once<0,false>", 4, 0)
L.fs_destroy(h)
""", tmp_path)


def test_batches_of_the_gpu_tests_run_the_kernels_they_are_meant_for(tmp_path):
    host_path.run(f"""
for dims, nb, voxel, fused, n, with_J, without in {large.CASES!r}:
    h, K = ctx(dims, nb=nb, init=VOXEL if voxel else BONE), 3 if voxel else nb
    assert precompute(h) == OK
    for kernel, kw in ((with_J, dict(slot=True)), (without, dict())):
        launched()
        assert solve(h, n, K, fused=fused, **kw) == OK
        assert kernel in [x.replace(" ", "") for x in names()], (kernel, n)
    # the largest batch of the kernels without queues is just below
    per, last = (294912, n - 1) if voxel and fused else (196608, None)
    if last is None:
        last = per // K
    assert solve(h, last, K, fused=fused) == OK and not [x for x in names() if x.startswith(("k_solve<", "k_solve_ws"))]
    L.fs_destroy(h)
""", tmp_path)


def test_arrays_that_overlap_go_to_the_kernels_that_write_last(tmp_path):
    # The kernels for small batches write the caller's arrays while other waves still read theirs; the others write
    # records, which a kernel of its own unpacks when the solve has ended.  A solve in place needs the latter.
    host_path.run("""
A, G = 0x300000000000, 1 << 30
p = ctypes.c_void_p
def kernels(h, N, K, xq=0, pose=1, x0=None, J0=None, v0=None, xc=5, conv=6, J=7, it=8, slot=9):
    launched()
    at = [None if a is None else p(A + int(a * G)) for a in (xq, pose, x0, J0, v0, xc, conv, J, it, slot)]
    assert L.fs_solve(h, *at[:2], ctypes.c_int64(N), K, *at[2:]) == OK
    return [x.split("<")[0] for x in names() if x.startswith("k_solve")]

small, large = (["k_solve_quad"], ["k_solve_once"]), ["k_solve_ws", "k_solve_unpack"]
h, K = ctx((64, 64, 16), P=2), 24
assert precompute(h) == OK
for N in (40, 5000):
    given = dict(x0=2, J0=3, v0=4)
    assert kernels(h, N, K) in small and kernels(h, N, K, **given) in small
    end = 12 * N * K / G                                     # of d_xc
    assert kernels(h, N, K, xq=5 + end) in small and kernels(h, N, K, xq=5 - 12 * N / G) in small       # side by side
    for kw in (dict(xq=5), dict(xq=5 + end - 16 / G), dict(xq=5 - 12 * N / G + 16 / G), dict(pose=5), dict(pose=6), dict(pose=7), dict(xq=8),
               dict(pose=9), dict(given, x0=5), dict(given, J0=7), dict(given, v0=6), dict(given, v0=8), dict(given, x0=7)):
        assert kernels(h, N, K, **kw) == large, (N, kw)
    assert kernels(h, N, K, pose=7, J=None) in small and kernels(h, N, K, **dict(given, v0=8, it=None)) in small
L.fs_destroy(h)
h = ctx((16, 16, 4), init=VOXEL)
assert precompute(h) == OK
assert kernels(h, 100, 3, pose=None) in small and kernels(h, 100, 3, pose=None, xq=5) == ["k_solve", "k_solve_unpack"]
L.fs_destroy(h)
""", tmp_path)


def test_exact_backward_takes_the_form_its_test_is_meant_for(tmp_path):
    host_path.run(f"""
p = Params(1e-5, 10.0, 50, 0, 1, 6, 5, 4, 3)
for dims, voxel, P, n, form in {exact.CASES!r}:
    p.init, K = (VOXEL, 3) if voxel else (BONE, 8)
    h = ctx(dims, nb=8, P=P, init=p.init)
    assert L.fs_set_params(h, ctypes.byref(p)) == OK and precompute(h) == OK and solve(h, n, K, slot=True) == OK
    for slot in (True, False):
        launched()
        assert grad(h, n, K, slot=slot) == OK
        assert f"k_grad_records<{{str(slot).lower()}},{{form}},1>" in [x.replace(" ", "") for x in names()], (dims, voxel, slot)
    L.fs_destroy(h)
""", tmp_path)


def test_pairs_on_grids_beyond_the_l2_are_handed_out_point_by_point(tmp_path):
    # In tiles of eight points the lines fetched for a point are gone when its next states come: a large batch on a large grid
    # (200 k points of 24 states on 128x128x32 nodes, 64 states, poses in any order) took 5 to 20 % longer.
    host_path.run(f"""
TILES, BY_POINT = 1, 2
def order(h, n, K, **kw):
    S.stub_clear_launches()
    assert solve(h, n, K, **kw) == OK
    return solve_params().point_major

for dims, P, nb, n, roots_only, positions in {large_grids.CASES!r}:
    h = ctx(dims, nb=nb, P=P)
    assert precompute(h) == OK
    assert (order(h, n, nb), order(h, n, nb, slot=True)) == (roots_only, positions), dims
    assert order(h, n, nb, fused=False, J=True) == TILES
    L.fs_destroy(h)
for dims, P, nb, n, expected in (((64, 64, 16), 1, 24, 1000000, TILES), ((128, 128, 32), 1, 24, 19000, TILES), ((128, 128, 32), 1, 24, 200000, BY_POINT),
                                 ((64, 64, 16), 8, 24, 60000, BY_POINT), ((61, 47, 13), 4, 24, 40003, TILES), ((80, 80, 20), 1, 64, 60000, BY_POINT)):
    h = ctx(dims, nb=nb, P=P)
    assert precompute(h) == OK and order(h, n, nb) == expected, (dims, n)
    L.fs_destroy(h)
""", tmp_path)


def test_an_order_that_is_asked_for_is_taken(tmp_path):
    host_path.run("""
def order(h, n, K, **kw):
    S.stub_clear_launches()
    assert solve(h, n, K, **kw) == OK
    return solve_params().point_major

calls = [dict(), dict(slot=True), dict(fused=False, J=True)]
for dims, n in (((16, 16, 4), 20000), ((64, 64, 16), 20000), ((128, 128, 32), 20000), ((128, 128, 32), 200000)):
    h = ctx(dims)
    assert precompute(h) == OK
    chosen = [order(h, n, 24, **kw) for kw in calls]
    assert set(chosen) <= {1, 2}
    assert L.fs_set_tuning(h, 0, 0, 0, 1, -1) == OK and [order(h, n, 24, **kw) for kw in calls] == [2, 2, 2]       # all states of a point
    assert L.fs_set_tuning(h, 0, 0, 0, 0, -1) == OK and [order(h, n, 24, **kw) for kw in calls] == [0, 0, 0]
    assert L.fs_set_tuning(h, 128, 0, 0, -1, -1) == OK and order(h, n, 24) == 0
    assert L.fs_set_tuning(h, 0, 0, 0, 2, -1) == E_ARG and L.fs_set_tuning(h, 0, 0, 0, -2, -1) == E_ARG
    L.fs_destroy(h)
""", tmp_path)


def test_share_of_the_chunks_that_is_dealt_out(tmp_path):
    host_path.run("""
def dealt(h, n, K, **kw):
    S.stub_clear_launches()
    assert solve(h, n, K, **kw) == OK
    return solve_params().dealt

for dims, P, init, expected in (((16, 16, 4), 1, BONE, 6), ((13, 15, 16), 1, BONE, 6), ((13, 15, 17), 1, BONE, 4), ((128, 128, 32), 1, BONE, 4), ((128, 128, 32), 2, BONE, 0),
                                ((16, 16, 4), 1, VOXEL, 6), ((64, 64, 16), 1, VOXEL, 6), ((128, 128, 32), 1, VOXEL, 6), ((128, 128, 32), 2, VOXEL, 0)):
    h, K = ctx(dims, P=P, init=init), 24 if init == BONE else 3
    assert precompute(h) == OK
    for kw in (dict(), dict(slot=True), dict(fused=False, J=True)):
        assert dealt(h, 400000 // K + 100000 * (init == VOXEL), K, **kw) == expected, (dims, P, init, kw)
    L.fs_destroy(h)
""", tmp_path)


def test_settings_until_they_are_set_are_those_the_header_states(tmp_path):
    host_path.run("""
for dims, P, init, refill, blocks in (((16, 16, 4), 1, BONE, 32, 3), ((16, 16, 4), 1, VOXEL, 32, 3), ((64, 64, 16), 1, BONE, 8, 3), ((64, 64, 16), 1, VOXEL, 8, 2),
                                      ((72, 72, 18), 1, BONE, 8, 2), ((128, 128, 32), 1, VOXEL, 8, 2), ((128, 128, 32), 2, BONE, 8, 2), ((128, 128, 32), 2, VOXEL, 24, 2)):
    h, K = ctx(dims, P=P, init=init), 24 if init == BONE else 3
    assert precompute(h) == OK
    for kw in (dict(), dict(slot=True), dict(fused=False, J=True)):
        S.stub_clear_launches()
        assert solve(h, 12000000 // K, K, **kw) == OK
        shape, at = (ctypes.c_uint * 7)(), [i for i in range(S.stub_launches()) if any(ctypes.string_at(S.stub_solve_params(i), 64))]
        S.stub_launch(at[0], shape)
        assert len(at) == 1 and shape[0] == blocks * 256, (dims, init, kw, shape[0])
        assert solve_params().refill_min == refill, (dims, init, kw)
    L.fs_destroy(h)
""", tmp_path)
