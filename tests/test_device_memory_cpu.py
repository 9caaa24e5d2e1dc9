"""Device memory of the library without a device: its host code, linked with a
HIP runtime that only keeps count (mock_hip.cpp).  A block must not be handed
on, or kept for that, while work that uses it has not been waited for."""
import ctypes
import os
import shutil
import subprocess

import pytest

from conftest import ROOT

CSRC = os.path.join(ROOT, "paper_2208_06290_amd", "csrc")
TESTS = os.path.dirname(os.path.abspath(__file__))
HIPCC = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"


@pytest.fixture(scope="module")
def built(tmp_path_factory):
    d = str(tmp_path_factory.mktemp("mock"))

    def run(*cmd):
        r = subprocess.run(cmd, cwd=d, capture_output=True, text=True)
        assert r.returncode == 0, r.stderr
        return r.stdout

    run(HIPCC, "-O1", "-std=c++17", "-fPIC", "--offload-host-only", "-w", "-I" + os.path.join(ROOT, "include"), "-c",
        os.path.join(CSRC, "hodlr_api.cpp"), "-o", "api.o")
    names = [w for w in run("nm", "-u", "api.o").split() if w.startswith("_ZN5hodlr") and "launch_" in w and
             "aca_own_launches" not in w]
    with open(os.path.join(d, "stubs.c"), "w") as f:
        f.write("int mock_launch(void*);\n" + "".join(f"int {n}(void* s) {{ return mock_launch(s); }}\n" for n in names))
    run("gcc", "-O1", "-fPIC", "-c", "stubs.c", "-o", "stubs.o")
    run("g++", "-O1", "-std=c++17", "-fPIC", "-c", os.path.join(TESTS, "mock_hip.cpp"), "-o", "mock.o")
    run("g++", "-shared", "-Wl,-Bsymbolic", "-Wl,-z,defs", "-o", "libmock.so", "api.o", "stubs.o", "mock.o", "-lpthread")
    return os.path.join(d, "libmock.so")


@pytest.fixture
def lib(built, tmp_path):
    copy = shutil.copy(built, tmp_path / "lib.so")  # its own pool and counters
    lib = ctypes.CDLL(str(copy))
    for f in ("mock_pending", "mock_graph_work", "mock_mallocs", "mock_frees"):
        getattr(lib, f).restype = ctypes.c_long
    lib.mock_used.restype = ctypes.c_size_t
    lib.mock_capacity.argtypes = [ctypes.c_size_t]
    lib.mock_fail_in.argtypes = [ctypes.c_long]
    lib.hodlr_destroy.argtypes = [ctypes.c_void_p]
    lib.hodlr_destroy.restype = None
    return lib


S1, S2 = ctypes.c_void_p(0x10), ctypes.c_void_p(0x20)  # streams
FAKE = 0x1000  # device addresses, never read


def _matrix(n, leaf, rank, dtype=0):
    from paper_2208_06290_amd import hodlr
    m = hodlr._Matrix()
    m.n, m.levels, m.dtype = n, (n // leaf).bit_length() - 1, dtype
    m.ranks = (ctypes.c_int32 * max(1, m.levels))(*[rank] * m.levels)
    m.D = m.U = m.V = FAKE
    m.ldd = m.ldu = m.ldv = n
    return m


def _factor(lib, m, stream):
    h = ctypes.c_void_p()
    st = lib.hodlr_factor(ctypes.byref(m), 0, 0, stream, ctypes.byref(h), None)
    return st, h


def _bytes(lib, n, leaf, rank):
    """What a factorization of this shape allocates."""
    before = lib.mock_used()
    st, h = _factor(lib, _matrix(n, leaf, rank), S1)
    assert st == 0
    return h, lib.mock_used() - before


def test_a_block_above_the_bound_leaves_the_kept_ones_alone(lib):
    small, nb = _bytes(lib, 4096, 64, 16)
    large, big = _bytes(lib, 1 << 20, 256, 32)
    assert nb < 1 << 30 and big > 4 << 30
    lib.hodlr_destroy(small)
    assert lib.mock_used() == nb + big  # kept
    lib.hodlr_destroy(large)
    assert lib.mock_used() < big, "a block larger than the bound goes straight back"
    assert lib.mock_used() >= nb, "and takes no other with it"
    count = lib.mock_mallocs()
    st, again = _factor(lib, _matrix(4096, 64, 16), S2)
    assert st == 0 and lib.mock_mallocs() == count
    lib.hodlr_destroy(again)


@pytest.mark.parametrize("dtype", [0, 3])  # FP64; complex, whose embedding the factorization owns
@pytest.mark.parametrize("launch", [0, 1, 2, 5, 9, 12])
def test_a_failed_refactorization_leaves_no_work_behind(lib, dtype, launch):
    m = _matrix(1024, 64, 8, dtype)
    st, h = _factor(lib, m, S1)
    assert st == 0
    lib.mock_fail_in(launch)
    assert lib.hodlr_refactor(h, ctypes.byref(m), S2, None) == -3
    lib.hodlr_destroy(h)  # its memory goes to the pool
    assert lib.mock_pending(S2) == 0


@pytest.mark.parametrize("dtype", [0, 3])
@pytest.mark.parametrize("launch", [0, 1, 3, 6, 12])
def test_a_failed_factorization_leaves_no_work_behind(lib, dtype, launch):
    lib.mock_fail_in(launch)
    st, h = _factor(lib, _matrix(1024, 64, 8, dtype), S2)
    assert st == -3 and not h
    assert lib.mock_pending(S2) == 0


@pytest.mark.parametrize("dtype", [0, 3])
def test_calls_that_allocate_are_refused_under_capture(lib, dtype):
    """As hipMalloc refuses then, so does the pool, whatever it holds."""
    m = _matrix(1024, 64, 8, dtype)
    ld = ctypes.c_int64(1024)
    X, Y = ctypes.c_void_p(FAKE), ctypes.c_void_p(2 * FAKE)

    def matvec(s):
        return lib.hodlr_matvec(ctypes.byref(m), 0, ctypes.c_int64(1), X, ld, Y, ld, s)

    st, h = _factor(lib, m, S1)
    assert st == 0 and matvec(S1) == 0
    st, other = _factor(lib, m, S1)
    lib.hodlr_destroy(other)  # the pool has blocks of every size needed
    lib.mock_record(S1, 1)
    assert matvec(S1) == -2
    assert _factor(lib, m, S1)[0] == -2
    assert lib.hodlr_solve(h, ctypes.c_int64(1), X, ld, None, S1, None) == -2  # no workspace of this stream yet
    assert lib.mock_graph_work() == 0  # nothing was recorded
    lib.mock_record(S1, 0)
    assert matvec(S1) == 0 and lib.hodlr_solve(h, ctypes.c_int64(1), X, ld, None, S1, None) == 0
    lib.mock_record(S1, 1)
    assert lib.hodlr_solve(h, ctypes.c_int64(1), X, ld, None, S1, None) == 0
    lib.mock_record(S1, 0)
    lib.hodlr_destroy(h)


@pytest.mark.parametrize("through", ["solve", "noalloc", "y_big"])
def test_release_waits_for_replays_of_recorded_calls(lib, through):
    """hipFree waited for the device; blocks that go to the pool must as well
    where a graph may still be replaying."""
    m = _matrix(1024, 64, 8)
    ld, X = ctypes.c_int64(1024), ctypes.c_void_p(FAKE)
    st, h = _factor(lib, m, S1)

    def call(n, stream):
        n = ctypes.c_int64(n)
        if through == "noalloc":
            return lib.hodlr_solve_noalloc(h, 0, n, X, ld, stream)
        if through == "y_big":
            return lib.hodlr_factors_y(h, X, ld, stream)
        return lib.hodlr_solve(h, n, X, ld, None, stream, None)

    assert st == 0 and call(1, S1) == 0
    lib.mock_record(S1, 1)
    assert call(1, S1) == 0
    lib.mock_record(S1, 0)
    assert lib.mock_graph_work() > 0
    if through == "solve":  # a larger workspace replaces the recorded one
        assert call(2, S1) == 0 and lib.mock_graph_work() == 0
        lib.mock_record(S1, 1)
        assert call(2, S1) == 0
        lib.mock_record(S1, 0)
    frees = lib.mock_frees()
    lib.hodlr_destroy(h)
    assert lib.mock_graph_work() == 0 and lib.mock_frees() == frees


def test_kept_blocks_are_given_back_on_request(lib):
    a, na = _bytes(lib, 4096, 64, 16)
    b, nb = _bytes(lib, 1024, 64, 8)
    lib.hodlr_destroy(a)
    assert lib.mock_used() == na + nb
    lib.hodlr_release_memory()
    assert lib.mock_used() == nb  # what has an owner stays
    lib.hodlr_destroy(b)
    lib.hodlr_release_memory()
    assert lib.mock_used() == 0


@pytest.mark.parametrize("call", ["solve", "adjoint", "noalloc", "grad", "y_big", "y_big complex", "logdet", "logdet_grad"])
def test_release_waits_for_the_last_call_on_every_stream(lib, call):
    st, h = _factor(lib, _matrix(1024, 64, 8, 3 if "complex" in call else 0), S1)
    n, ld, X = ctypes.c_int64(2), ctypes.c_int64(1024), ctypes.c_void_p(FAKE)
    d = ctypes.c_double()
    assert st == 0
    for s in (S1, S2):
        assert 0 == {"solve": lambda: lib.hodlr_solve(h, n, X, ld, None, s, None),
                     "adjoint": lambda: lib.hodlr_solve_adjoint(h, n, X, ld, None, s, None),
                     "noalloc": lambda: lib.hodlr_solve_noalloc(h, 1, n, X, ld, s),
                     "grad": lambda: lib.hodlr_grad(h, n, X, ld, X, ld, X, X, X, s),
                     "y_big": lambda: lib.hodlr_factors_y(h, X, ld, s),
                     "y_big complex": lambda: lib.hodlr_factors_y(h, X, ld, s),
                     "logdet": lambda: lib.hodlr_logdet(h, ctypes.byref(d), ctypes.byref(d), s),
                     "logdet_grad": lambda: lib.hodlr_logdet_grad(h, X, X, X, s)}[call]()
    lib.hodlr_destroy(h)
    assert lib.mock_pending(S2) == 0
    if call != "noalloc":  # one scratch, whose calls the caller orders: the last one is waited for
        assert lib.mock_pending(S1) == 0
