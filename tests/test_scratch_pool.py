"""Device memory that the library keeps between step-level calls, seen from a
stand-in for the HIP runtime (fake_hip.cpp: host memory up to a limit, launches
that do nothing): it gives way to every other allocation of the library."""
import os
import shutil
import subprocess
import sys
import textwrap

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_1212_3660_amd", "libshk.so")

PRELUDE = """
import ctypes as C, sys
import numpy as np
fake = C.CDLL(sys.argv[1], mode=C.RTLD_GLOBAL)
L = C.CDLL(sys.argv[2])
fake.fake_live.restype = C.c_size_t
fake.fake_limit.argtypes = [C.c_size_t]
NONE = C.c_size_t(-1).value

def ptr(a):
    return a.ctypes.data_as(C.c_void_p)

def problem(nx=8, ny=8):
    K, p = np.full(nx * ny, 1e-5), C.c_void_p()
    rc = L.shk_problem_create_fv2d(C.c_int(nx), C.c_int(ny), ptr(K), C.c_double(1e-5),
                                   C.c_double(1.0), C.byref(p))
    return rc, p

def destroy(p):
    L.shk_problem_destroy(p)

def least_squares(nf, k=20):
    # a step-level call that needs no problem; its scratch grows with the shifts
    a = [np.zeros(s, complex) for s in ((k + 1) * k, k, nf, nf * k)]
    return L.shk_shifted_lsq(k, ptr(a[0]), ptr(a[1]), nf, ptr(a[2]), C.c_double(1.0), ptr(a[3]),
                             ptr(np.zeros(nf * k)), 0)

def orthogonalize(n, k=2):
    V, w, h = np.zeros((k + 1, n), complex), np.zeros(n, complex), np.zeros(k + 1, complex)
    return L.shk_orthogonalize(C.c_longlong(n), 1, k, ptr(V), ptr(w), ptr(h), 0, 0, None)
"""


@pytest.fixture(scope="module")
def fake(tmp_path_factory):
    if not os.path.exists(LIB) or not shutil.which("g++"):
        pytest.skip("needs the built library and g++")
    out = str(tmp_path_factory.mktemp("fake") / "libfake_hip.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-pthread", "-o", out,
                    os.path.join(ROOT, "tests", "fake_hip.cpp")], check=True)
    return out


def _run(fake, body):
    r = subprocess.run([sys.executable, "-c", PRELUDE + textwrap.dedent(body), fake, LIB], capture_output=True,
                       text=True, timeout=100)
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-2000:]


# Each allocation gets exactly the memory that the kept blocks hold beside what
# is in use: it succeeds only after they are given back.
@pytest.mark.parametrize("what", ["grid", "csr", "solve", "server"])
def test_kept_blocks_give_way(fake, what):
    _run(fake, """
        WHAT = %r
        rc, p = problem()
        assert rc == 0
        used = fake.fake_live()
        assert least_squares(1000) == 0
        kept = fake.fake_live() - used
        assert kept > 2 << 20, kept
        fake.fake_limit(used + kept)
        if WHAT == "grid":
            rc, q = problem(150, 150)
        elif WHAT == "csr":
            n = 20000
            rp, col, val, md = np.arange(n + 1, dtype=np.int32), np.arange(n, dtype=np.int32), np.ones(n), np.ones(n)
            q = C.c_void_p()
            rc = L.shk_problem_create_csr(n, *map(ptr, (rp, col, val, md)), C.byref(q))
        elif WHAT == "server":
            q = C.c_void_p()
            rc = L.shk_server_create(C.c_size_t(kept & ~255), 1, None, C.byref(q))
            if rc == 0:
                L.shk_server_destroy(q)
        else:
            class Params(C.Structure):   # shk_params of include/shk.h
                _fields_ = [(f, C.c_int) for f in ("m_restart", "max_restarts", "max_refine", "inner_maxit")] + [
                    ("tol", C.c_double), ("eps_inner", C.c_double), ("n_tau", C.c_int), ("tau_seq", C.c_void_p),
                    ("rest", C.c_char * 256)]
            prm = Params()
            L.shk_params_default(C.byref(prm))
            tau, sigma = np.array([0.1j]), np.array([0.1j, 0.2j])
            prm.m_restart, prm.max_restarts, prm.max_refine, prm.inner_maxit, prm.n_tau = 1, 0, 0, 1, 1
            prm.tau_seq = tau.ctypes.data
            need = C.c_size_t()
            assert L.shk_workspace_bytes(p, C.byref(prm), 2, 1, C.byref(need)) == 0
            fake.fake_limit(used + max(kept, need.value) + (1 << 10))
            b, x, st = np.ones(64, complex), np.zeros((2, 64), complex), np.zeros(4096, np.uint8)
            rc = L.fgmres_sh_solve(p, C.byref(prm), 2, ptr(sigma), 1,
                                   ptr(b), ptr(x),
                                   ptr(st), None, C.c_size_t(0), None, 1)
        assert rc == 0, rc
        fake.fake_limit(NONE)
        # a request that fails all the same leaves no error behind for the next call
        fake.fake_limit(fake.fake_live())
        L.shk_server_create.restype = C.c_int
        assert L.shk_server_create(C.c_size_t(1 << 30), 1, None, C.byref(C.c_void_p())) == -2
        fake.fake_limit(NONE)
        assert least_squares(10) == 0
    """ % what)


def test_nothing_is_kept_without_a_problem(fake):
    _run(fake, """
        assert least_squares(1000) == 0
        assert fake.fake_live() == 0, fake.fake_live()
        rc, p = problem()
        used = fake.fake_live()
        assert least_squares(1000) == 0 and fake.fake_live() > used
        destroy(p)
        assert fake.fake_live() == 0, fake.fake_live()
        assert least_squares(1000) == 0
        assert fake.fake_live() == 0, fake.fake_live()
    """)


def test_a_release_holds_up_no_other_call(fake):
    """hipFree waits for the work on the device: while one thread stands in it
    with the blocks of the last problem, another thread's call goes through."""
    _run(fake, """
        import threading
        rc, p = problem()
        assert least_squares(1000) == 0
        fake.fake_gate_arm()       # taken by the first hipFree: a kept block's
        t = threading.Thread(target=destroy, args=(p,))
        t.start()
        assert fake.fake_gate_entered()
        assert least_squares(300) == 0
        assert fake.fake_gate_open() == 1
        t.join()
        assert fake.fake_live() == 0
    """)


def test_giving_a_block_back_needs_no_host_memory(fake):
    """It happens in a destructor, where an exception ends the process."""
    _run(fake, """
        rc, p = problem()
        fake.fake_no_new(1)
        rc = orthogonalize(500)
        fake.fake_no_new(0)
        assert rc == 0
    """)
