"""Host code of the library on a stub runtime (host_path.py): what it launches and what it answers when memory runs out."""
import host_path


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


def test_precompute_that_runs_out_of_memory_leaves_the_old_grid_whole(tmp_path):
    # The words that the scan of the correspondence build needs grow on demand, and are gone when growing them failed
    # in another call.  fs_precompute has to ask for them before it launches anything: with a new transform grid beside
    # the candidates of the old one the context would answer fs_solve with a mixture of both.
    host_path.run("""
h, n, K = ctx((64, 64, 16), init=VOXEL), 1 << 23, 3
assert precompute(h) == OK and solve(h, n, K) == OK
launched()
look = 0
for i in range(8):                          # a larger solve, its i-th allocation fails; one of them is the scan's
    S.stub_fail_allocation(i)
    st = solve(h, n * (i + 2), K)
    S.stub_fail_allocation(-1)
    assert st in (OK, E_ALLOC)
    if b"(scan)" in L.fs_last_error(h):
        look = 1
        break
assert look
launched()
S.stub_fail_allocation(0)
assert precompute(h) == E_ALLOC
assert launched() == [], "half a pose"
S.stub_fail_allocation(-1)
assert precompute(h) == OK and solve(h, n, K) == OK
L.fs_destroy(h)
assert S.stub_bad_frees() == 0 and S.stub_live_blocks() == 0
""", tmp_path)
