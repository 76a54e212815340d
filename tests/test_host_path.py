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
