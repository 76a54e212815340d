"""The library's host code without a GPU: libfastsnarf.so on top of the runtime of host_stub.c, which makes addresses up,
records kernel launches instead of running them, and fails allocations on request.

The stub has to be found before the real runtime, so this runs in a child process (`run`) that loads it first and imports
no torch.  In the child: `ctx(...)`, `buf()`, `launched()`, `L` (the library), `S` (the stub)."""
import ctypes
import os
import re
import subprocess
import sys

HERE = os.path.dirname(os.path.abspath(__file__))
LIB = os.path.join(os.path.dirname(HERE), "paper_2211_15601_amd", "csrc", "libfastsnarf.so")


def run(code, tmp_path):
    """Executes `code` in a child process on the stub runtime; fails with its output if it fails."""
    stub = os.path.join(str(tmp_path), "host_stub.so")
    subprocess.check_call(["gcc", "-shared", "-fPIC", "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                           os.path.join(HERE, "host_stub.c"), "-o", stub])
    env = dict(os.environ, FS_HOST_STUB=stub, PYTHONPATH=HERE)
    r = subprocess.run([sys.executable, "-c", "from host_path import *\n" + code + "\nprint('CHILD-OK')"], env=env,
                       capture_output=True, text=True, timeout=120)
    assert r.returncode == 0 and "CHILD-OK" in r.stdout, (r.stdout + r.stderr)[-3000:]


# ---- in the child ----
OK, E_ARG, E_SHAPE, E_STATE, E_ALLOC, E_DEVICE, E_UNSUPPORTED = range(7)
BONE, VOXEL = 0, 1


class Desc(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int32) for n in ("nx", "ny", "nz", "nb", "P")] + [("lo", ctypes.c_float * 3), ("hi", ctypes.c_float * 3)]


class Params(ctypes.Structure):
    _fields_ = [("tol", ctypes.c_float), ("div", ctypes.c_float)] + [(n, ctypes.c_int32) for n in ("iters", "init", "grad", "cx", "cy", "cz", "ck")]


class SolveP(ctypes.Structure):
    """what a solve kernel with queues is told (fs_kernels.hpp)"""
    _fields_ = [(n, ctypes.c_int64) for n in ("N", "total")] + [(n, ctypes.c_int32) for n in ("chunk", "refill_min", "max_iters")] + \
               [(n, ctypes.c_float) for n in ("tol2", "div2")] + \
               [(n, ctypes.c_int32) for n in ("K", "point_major", "ki", "spin_limit", "xcd_ranges", "dealt", "prefetch")]


if "FS_HOST_STUB" in os.environ:
    S = ctypes.CDLL(os.environ["FS_HOST_STUB"], mode=ctypes.RTLD_GLOBAL)
    S.stub_launch.restype = ctypes.c_char_p
    S.stub_solve_params.restype = ctypes.c_void_p
    L = ctypes.CDLL(LIB)
    L.fs_last_error.restype = ctypes.c_char_p


def ctx(dims, nb=24, P=1, init=BONE, ck=3, corr=(6, 5, 4)):
    d = Desc(*dims, nb, P, (ctypes.c_float * 3)(-1, -1, -1), (ctypes.c_float * 3)(1, 1, 1))
    p = Params(1e-5, 10.0, 50, init, 0, *corr, ck)
    h = ctypes.c_void_p()
    assert L.fs_create(ctypes.byref(d), ctypes.byref(p), None, ctypes.byref(h)) == OK
    return h


def buf(i=0):
    """an address that is accepted as device memory (nothing reads or writes it), 64 GiB of it for every i"""
    return ctypes.c_void_p(0x300000000000 + (i << 36))


def precompute(h):
    return L.fs_precompute(h, buf(), buf())


def solve(h, N, K, fused=True, J=False, slot=False):
    init = (None, None, None) if fused else (buf(2), buf(3), buf(4))
    return L.fs_solve(h, buf(0), buf(1), ctypes.c_int64(N), K, *init, buf(5), buf(6), buf(7) if J else None, buf(8), buf(9) if slot else None)


def grad(h, N, K, slot=False):
    b = buf()
    return L.fs_grad(h, b, b, b, b, b, b, ctypes.c_int64(N), K, b if slot else None, b, b, b)


def launched():
    """what was launched since the last call: [(kernel with its template arguments, grid, block, bytes of dynamic LDS)]"""
    demangle = ctypes.CDLL("libstdc++.so.6")["__cxa_demangle"]
    demangle.restype, demangle.argtypes = ctypes.c_char_p, [ctypes.c_char_p] + 3 * [ctypes.c_void_p]
    out, shape = [], (ctypes.c_uint * 7)()
    for i in range(S.stub_launches()):
        name = demangle(S.stub_launch(i, shape), None, None, None).decode()
        m = re.match(r"(?:void )?fs::(\w+(?:<[^(]*>)?)\(", name)
        out.append((m.group(1), tuple(shape[:3]), tuple(shape[3:6]), shape[6]))
    S.stub_clear_launches()
    return out


def solve_params():
    """of the one solve kernel with queues launched since the last call"""
    at = [S.stub_solve_params(i) for i in range(S.stub_launches())]
    (p,) = [SolveP.from_buffer_copy(ctypes.string_at(a, 64)) for a in at if any(ctypes.string_at(a, 64))]
    S.stub_clear_launches()
    return p


def names():
    return [l[0] for l in launched()]
