"""What the library launches, without a GPU: the host code of libgpspca.so runs
against a stub of the HIP runtime (hip_stub.cpp) that records every launch.
Each scenario is a function of this file run in a child process of its own,
which loads the stub before the library and never imports torch."""
import ctypes
import importlib.util
import os
import subprocess
import sys

import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)


def _module(name, *path):
    spec = importlib.util.spec_from_file_location(name, os.path.join(ROOT, *path))
    mod = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(mod)
    return mod


@pytest.fixture(scope="module")
def stub(tmp_path_factory):
    hipcc = _module("gpspca_build", "paper_1312_6182_amd", "build.py").hipcc()
    so = str(tmp_path_factory.mktemp("stub") / "libhipstub.so")
    subprocess.run([hipcc, "-x", "hip", "--offload-host-only", "-std=c++17", "-O1", "-shared",
                    "-fPIC", "-I", os.path.join(ROOT, "include"),
                    os.path.join(HERE, "hip_stub.cpp"), "-o", so], check=True, capture_output=True)
    return so


def _child(stub, scenario, **env):
    r = subprocess.run([sys.executable, os.path.abspath(__file__), scenario, stub],
                       capture_output=True, text=True, timeout=120, env={**os.environ, **env})
    assert r.returncode == 0, r.stdout[-2000:] + r.stderr[-4000:]


class Lib:
    """The library on the stub; pointers to device memory are made up."""

    DATA, WS, OUT = 1 << 40, 1 << 44, 1 << 46

    def __init__(self, stub):
        self.stub = ctypes.CDLL(stub, mode=ctypes.RTLD_GLOBAL)
        self.stub.stub_log.restype = ctypes.c_size_t
        self.L = _module("gpspca_lib", "paper_1312_6182_amd", "_lib.py")
        self.lib = self.L.load()
        self.result(1)

    def device(self, cus, masked=0):
        """CUs of the device (the library reads them once), and how many of them are
        closed to streams."""
        self.stub.stub_device(cus, masked)

    def result(self, n_iter, status=1, abort=0):
        self.stub.stub_result(n_iter, status, abort)

    def launches(self):
        """(kernel name, (gx, gy, gz), threads, LDS bytes, stream, quantized columns)"""
        n = self.stub.stub_log(None, ctypes.c_size_t(0))
        buf = ctypes.create_string_buffer(n + 1)
        self.stub.stub_log(buf, ctypes.c_size_t(n + 1))
        out = []
        for line in buf.value.decode().splitlines():
            f = line.split()
            out.append((f[0], tuple(int(v) for v in f[1:4]), int(f[4]), int(f[5]), f[6], int(f[7])))
        return out

    def names(self):
        return [k[0] for k in self.launches()]

    def matrix(self, p, n, dtype=0, odd=False):
        M = self.L.Matrix()
        pad = (4, 8, 16)[dtype]
        M.data, M.p, M.n, M.dtype = self.DATA, p, n, dtype
        M.lda = p | 1 if odd else (p + pad - 1) // pad * pad
        M.col_scale = 1 << 45 if dtype == self.L.F8E4M3 else None
        return M

    def solve(self, M, m=1, form=None, max_iter=1, tol=0.0, stream=None):
        form = (self.L.SL1 if m == 1 else self.L.BL1) if form is None else form
        nb = self.lib.gpspca_workspace_bytes(ctypes.byref(M), form, m, max_iter)
        assert nb > 0, self.lib.gpspca_last_error()
        nit = ctypes.c_int(0)
        trace = (ctypes.c_double * max_iter)()
        return self.lib.gpspca_solve(ctypes.byref(M), form, m, 0.1, None, None, tol, max_iter,
                                     self.WS, nb, stream, self.OUT, self.OUT, self.OUT, trace,
                                     ctypes.byref(nit))

    def autotune(self, M, m=1, form=None, times=(1.0, 1.0)):
        """(configurations timed, description of the chosen one)"""
        form = (self.L.SL1 if m == 1 else self.L.BL1) if form is None else form
        self.stub.stub_times(ctypes.c_float(times[0]), ctypes.c_float(times[1]))
        size = (self.lib.gpspca_path_workspace_bytes(ctypes.byref(M), m, 4)
                if form == self.L.SL1 and m > 1 else
                self.lib.gpspca_workspace_bytes(ctypes.byref(M), form, m, 4))
        timed, desc = ctypes.c_int(0), ctypes.create_string_buffer(128)
        rc = self.lib.gpspca_autotune(ctypes.byref(M), form, m, 0.1, self.OUT, 3, self.WS, size,
                                      None, ctypes.byref(timed), None, desc, 128)
        assert rc == 0, self.lib.gpspca_last_error()
        return timed.value, desc.value.decode()

    def multistart(self, M, m, max_iter=1):
        nb = self.lib.gpspca_path_workspace_bytes(ctypes.byref(M), m, max_iter)
        nit, st = (ctypes.c_int * m)(), (ctypes.c_int * m)()
        return self.lib.gpspca_solve_multistart(ctypes.byref(M), self.L.SL1, m, 0.1, 0.0, max_iter,
                                                self.WS, nb, None, self.OUT, self.OUT, self.OUT,
                                                None, nit, st)


def _check_limits(case, launches):
    assert launches, case
    for name, grid, threads, lds, _, _ in launches:
        assert all(1 <= g and g * threads < 1 << 32 for g in grid[:1]), (case, name, grid, threads)
        assert grid[1] < 1 << 16 and grid[2] < 1 << 16, (case, name, grid)
        assert 1 <= threads <= 1024 and 0 <= lds <= 160 * 1024, (case, name, threads, lds)


def child_launch_limits(lib):
    """Every launch of a solve within the limits of the hardware, from one row and
    column to matrices that fill the memory of a GPU."""
    shapes = [(1, 1), (1, 1000), (4, 100000), (100, 1000), (1000, 10000), (1900, 64), (9000, 50),
              (10000, 100000), (100000, 1000), (1 << 20, 64),
              (1000, 34_000_000), (1000, 60_000_000), (16, (1 << 30) - 64), (40, 900_000_000)]
    for p, n in shapes:
        for dtype in (0, 1, 2):
            if p * n * (4, 2, 1)[dtype] > 280 << 30:
                continue
            M = lib.matrix(p, n, dtype)
            for m in (1, 2, 5, 8, 16, 64):
                if m > min(p, n) or 4 * m * n > 200 << 30:
                    continue
                case = (p, n, dtype, m)
                assert lib.solve(M, m) >= 0, (case, lib.lib.gpspca_last_error())
                _check_limits(case, lib.launches())
                if m <= 16:
                    assert lib.multistart(M, m) >= 0, (case, "multistart")
                    _check_limits((case, "multistart"), lib.launches())


def test_launch_limits(stub):
    _child(stub, "launch_limits")


def child_quantize_limits(lib):
    """The quantizer's launches cover every column, each within the 2^32 work
    items of a dimension (a grid of 2^24 workgroups of 256 threads is too large)."""
    for p, n in ((3, 50_000_000), (2560, 100), (2561, 20_000_000), (10240, (1 << 24) - 1),
                 (10240, 1 << 24), (10241, 5_000_000), (40961, 1_000_000)):
        M = lib.matrix(p, n)
        for to, ld in ((1, (p + 7) // 8 * 8), (2, (p + 15) // 16 * 16)):
            assert lib.lib.gpspca_quantize(ctypes.byref(M), to, lib.WS, ld, lib.OUT, None) == 0
            launches = lib.launches()
            _check_limits((p, n, to), launches)
            assert sum(k[5] for k in launches) == n, (p, n, launches)


def test_quantize_limits(stub):
    _child(stub, "quantize_limits")


def _small(lib):
    """Workgroups of the persistent kernel in the launches so far (none: [])."""
    return [k[1][0] for k in lib.launches() if "k_small" in k[0]]


# persistent solves that take 8, 13, 50 and 64 workgroups on a whole GPU
SMALL = [(100, 1000, 8), (150, 1600, 13), (400, 4000, 50), (16, 60000, 64)]


def child_few_cus(lib):
    """A device of 32 CUs (one XCD of a partitioned GPU) takes solves of up to half
    as many workgroups."""
    lib.device(32)
    for p, n, nb in SMALL:
        assert lib.solve(lib.matrix(p, n), 1, max_iter=4) >= 0
        assert _small(lib) == ([nb] if nb <= 16 else []), (p, n)


def child_masked_stream(lib):
    """On a stream that is kept off some CUs the XCDs may hold fewer workgroups than
    the admission counts on: the passes are separate launches there."""
    lib.device(256)
    for p, n, nb in SMALL:
        M = lib.matrix(p, n)
        assert lib.solve(M, 1, max_iter=4) >= 0 and _small(lib) == [nb]
        lib.device(256, masked=200)
        assert lib.solve(M, 1, max_iter=4) >= 0 and _small(lib) == []
        lib.device(256)
    M = lib.matrix(20, 100)          # one workgroup waits for nobody
    lib.device(256, masked=200)
    assert lib.solve(M, 1, max_iter=4) >= 0 and _small(lib) == [1]


def child_run_out(lib):
    """A wait that ran out is not waited for again at once: the passes run as
    launches, and so do the next 64 solves of that size or another; a second
    run-out in a row doubles that, a solve that ends well ends it.  A limit longer
    than the one that ran out is tried."""
    M, other = lib.matrix(100, 1000), lib.matrix(150, 1600)

    def solve(A=M, abort=0):
        lib.result(1, abort=abort)
        assert lib.solve(A, 1, max_iter=4) >= 0
        names = lib.names()
        return sum("k_small" in k for k in names), sum("k_pass_m1" in k for k in names)

    assert solve() == (1, 0)
    for quiet in (64, 128, 256):
        assert solve(abort=1) == (1, 4)
        for i in range(quiet):
            assert solve(other if i % 2 else M) == (0, 4), (quiet, i)
    assert solve() == (1, 0) and solve() == (1, 0)
    assert solve(abort=1) == (1, 4)
    assert solve() == (0, 4)
    os.environ["GPSPCA_SMALL_WAIT"] = str(1 << 40)
    assert solve() == (1, 0)


def child_queued(lib):
    """Solves that wait behind long work of their own streams keep nobody from
    starting: four of 64 workgroups, whose streams move on only when a fifth one on
    an idle stream has ended."""
    import threading
    ended = threading.Event()
    streams = [0x10000 * (i + 1) for i in range(4)]
    wait = ctypes.CFUNCTYPE(None, ctypes.c_void_p)(
        lambda st: st in streams and (ended.wait(60) or os._exit(3)))
    lib.stub.stub_on_sync(wait)
    M = lib.matrix(16, 60000)
    rc = [None] * 5

    def run(i, stream):
        rc[i] = lib.solve(M, 1, max_iter=4, stream=stream)

    ts = [threading.Thread(target=run, args=(i, st)) for i, st in enumerate(streams)]
    for t in ts:
        t.start()
        t.join(0.3)          # it launches its passes, or waits
        assert t.is_alive()
    last = threading.Thread(target=run, args=(4, None), daemon=True)
    last.start()
    last.join(20)
    assert not last.is_alive(), "an idle stream's solve waits for queued ones"
    ended.set()
    for t in ts:
        t.join()
    assert min(rc) >= 0 and _small(lib) == [64] * 5


def child_special_streams(lib):
    """The handles of the legacy and the per-thread default stream (1 and 2) are no
    addresses: the query of a stream's CU mask must not be given them."""
    for stream in (None, 1, 2):
        assert lib.solve(lib.matrix(100, 1000), 1, max_iter=4, stream=stream) >= 0
        assert _small(lib) == [8]


@pytest.mark.parametrize("scenario", ["few_cus", "masked_stream", "run_out", "queued",
                                      "special_streams"])
def test_persistent_solves_need_their_cus(stub, scenario):
    _child(stub, scenario)


def child_autotune(lib):
    """The autotuner times the persistent kernel of a small matrix beside the
    launches and later solves take what won; a tuned default is no reason to
    leave the kernel."""
    for m, form, p, n in ((1, None, 100, 1000), (1, None, 400, 4000), (5, None, 200, 2000),
                          (4, lib.L.SL1, 100, 1000)):
        M = lib.matrix(p, n)

        def kernels():
            lib.launches()
            rc = lib.multistart(M, m, 4) if form is not None else lib.solve(M, m, max_iter=4)
            assert rc >= 0
            return sum("k_small" in k for k in lib.names())

        assert kernels() == 1
        timed, desc = lib.autotune(M, m, form, times=(1.0, 2.0))
        assert timed >= 2 and desc.startswith("k_small workgroups="), (timed, desc)
        assert sum("k_small" in k for k in lib.names()) == 2     # untimed, timed
        assert kernels() == 1
        timed, desc = lib.autotune(M, m, form, times=(1.05, 1.0))
        assert desc.startswith("k_small")    # launches have their own cost per solve
        timed, desc = lib.autotune(M, m, form, times=(2.0, 1.0))
        lib.launches()
        assert "k_small" not in desc and kernels() == 0, (m, form, desc)
        lib.lib.gpspca_autotune_clear()
        assert kernels() == 1
    # no persistent kernel: as many configurations as there are correlation kernels
    assert lib.autotune(lib.matrix(5000, 50000))[0] == 1
    lib.result(1, abort=1)       # it gave up: it is not chosen
    assert "k_small" not in lib.autotune(lib.matrix(100, 1000), times=(1.0, 2.0))[1]


def test_autotune_of_small_matrices(stub):
    _child(stub, "autotune")


def child_short_columns(lib):
    """The kernels that short columns take: what was measured fastest for them."""
    def norms(p, dtype):
        assert lib.lib.gpspca_column_norms(ctypes.byref(lib.matrix(p, 1000, dtype)), lib.OUT,
                                           None) == 0
        return "short" in lib.names()[0]

    for dtype, last in ((0, 256), (1, 512), (2, 1024)):
        assert norms(last, dtype) and not norms(last + 1, dtype)

    def corr(p, n, m, dtype):
        assert lib.solve(lib.matrix(p, n, dtype), m, max_iter=1) >= 0
        names = lib.names()
        return [k for k in ("k_corr_sh", "k_corr_qw", "k_small") if any(k in x for x in names)]

    for dtype in (1, 2):
        assert corr(64, 200000, 5, dtype) == ["k_corr_qw"]
        assert corr(256, 40000, 16, dtype) == ["k_corr_qw"]
        assert corr(512, 200000, 17, dtype) == ["k_corr_qw"]
        assert corr(600, 60000, 16, dtype) == ["k_corr_sh"]
        assert corr(2000, 20000, 32, dtype) == ["k_corr_sh"]
    assert corr(400, 8000, 16, 1) == ["k_corr_sh"]


def test_short_columns(stub):
    _child(stub, "short_columns")


def child_workspace(lib):
    """A step takes the workspace that a solve of one pass takes: where only the
    default correlation's buffers are too large, the leaner one runs."""
    ENOMEM = lib.L.ENOMEM
    for p, n, dtype, m, odd in ((1001, 20001, 0, 12, True), (1003, 30000, 0, 64, False),
                                (2000, 30000, 1, 16, False), (4000, 40000, 2, 8, False)):
        M = lib.matrix(p, n, dtype, odd)

        def step(nb):
            return lib.lib.gpspca_step(ctypes.byref(M), lib.L.BL1, m, 0.1, None, lib.OUT, lib.WS,
                                       nb, None, lib.OUT, None, None, None)

        def solve(nb):
            return lib.lib.gpspca_solve(ctypes.byref(M), lib.L.BL1, m, 0.1, None, None, 0.0, 1,
                                        lib.WS, nb, None, lib.OUT, None, None, None, None)

        lo, hi = 0, lib.lib.gpspca_workspace_bytes(ctypes.byref(M), lib.L.BL1, m, 1) // 256
        assert solve(256 * hi) >= 0 and step(256 * hi) >= 0
        while hi - lo > 1:
            mid = (lo + hi) // 2
            lo, hi = (lo, mid) if solve(256 * mid) >= 0 else (mid, hi)
        assert step(256 * hi) >= 0, (p, n, m)
        assert solve(256 * lo) == step(256 * lo) == ENOMEM


def test_step_and_solve_take_the_same_workspace(stub):
    _child(stub, "workspace")


if __name__ == "__main__":
    globals()["child_" + sys.argv[1]](Lib(sys.argv[2]))
