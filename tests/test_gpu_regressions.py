"""Faults that were found in the kernels and their dispatch, one test each."""
import ctypes

import numpy as np
import pytest
import torch

import oracle as O
from workloads import generators as W

from _util import fp32_round, pick_gamma, rel, to_device, x_to_device

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("lda", [104, 101], ids=["aligned", "odd"])
@pytest.mark.parametrize("row", [0, 96, 99, 100], ids=["first", "last_quad", "last_quad_end", "tail"])
@pytest.mark.parametrize("m", [8, 32, 40])
def test_infinity_in_the_last_slots_is_seen(gpu, m, row, lda, monkeypatch):
    """k_corr_sh repeats a column's last full slot against zeros of X in its last
    stage (101 rows: 25 slots of 16 or 8 a stage); an infinity there must make
    the objective non-finite as it does in any other row."""
    monkeypatch.setenv("GPSPCA_CORR_KERNEL", "sh")
    p, n = 101, 200
    A = W.gaussian(p, n, 5)
    A[row, 7] = np.inf
    X = fp32_round(W.random_orthonormal(p, m, 8))
    assert (X[row] != 0).all()
    with pytest.raises(gpu.GpspcaError) as e:
        gpu.step(to_device(A, lda=lda), O.BL1, x_to_device(X), 0.5)
    assert e.value.code == gpu.ENONFINITE


def _correlation_error(gpu, Ad, X, ref):
    """Relative error of y = A^T X (gamma = 0: S is y) in the 2-norm."""
    d = gpu.step(Ad, O.BL1, X, 0.0).S.double() - ref
    return float(d.norm() / ref.norm())


# sizes with at least 1e5 correlations: the 2-norm of their errors is then known to
# well under 5%
@pytest.mark.parametrize("m", [5, 16, 32, 64])
@pytest.mark.parametrize("p,n", [(101, 20000), (399, 20000), (401, 20000), (1001, 20000),
                                 (5003, 20000)])
def test_unaligned_columns_keep_the_vector_kernels_accuracy(gpu, p, n, m, monkeypatch):
    """FP32 columns at odd leading dimensions: k_corr_sh is no further from FP64
    than the vector-ALU kernel, whose lanes add p / 64 rows each (5% for the
    samples)."""
    gen = torch.Generator(device="cuda").manual_seed(p + m)
    A = torch.randn((n, p), device="cuda", generator=gen).t()
    X = x_to_device(fp32_round(W.random_orthonormal(p, m, 9)))
    ref = A.t().double() @ X.double()
    err = {}
    for k in ("sh", "valu"):
        monkeypatch.setenv("GPSPCA_CORR_KERNEL", k)
        err[k] = _correlation_error(gpu, A, X, ref)
    print(f"\n[accuracy] p={p} m={m} {err}", flush=True)
    assert err["sh"] <= 1.05 * err["valu"]


def test_64_components_keep_the_accuracy_of_short_chains(gpu, monkeypatch):
    """Aligned FP32 with 64 components: an accumulator through all 10000 rows is off
    by 1.6e-6; with totals every 32 to 256 rows the rounding of the totals and of the
    products in between stays below a third of that."""
    p, n, m = 10000, 6000, 64
    gen = torch.Generator(device="cuda").manual_seed(4)
    A = torch.randn((n, p), device="cuda", generator=gen).t()
    X = x_to_device(fp32_round(W.random_orthonormal(p, m, 9)))
    monkeypatch.setenv("GPSPCA_CORR_KERNEL", "sh")
    assert _correlation_error(gpu, A, X, A.t().double() @ X.double()) <= 5e-7


def _two_passes64(A, X0, gamma, polar):
    """X_1 and the unit-norm Z of the second pass of an L1 solve, in FP64."""
    def soft(X):
        Y = A.t() @ X
        return torch.sign(Y) * (Y.abs() - gamma).clamp_min(0.0)

    G = A @ soft(X0)
    if polar:
        w, V = torch.linalg.eigh(G.t() @ G)
        X = G @ (V / w.sqrt()) @ V.t()
    else:
        X = G / G.norm(dim=0)
    S = soft(X)
    return X, S / S.norm(dim=0)


@pytest.mark.parametrize("pad", [0, 1], ids=["aligned", "odd"])
@pytest.mark.parametrize("kind,m", [("SL1", 1), ("BL1", 2), ("BL1", 5), ("BL1", 8), ("multi", 4),
                                    ("multi", 16)])
@pytest.mark.parametrize("p,n", [(100, 1000), (200, 2000), (400, 4000), (400, 100), (1200, 600)])
def test_persistent_solves_keep_the_launches_accuracy(gpu, p, n, kind, m, pad, monkeypatch):
    """Two passes of k_small are no further from FP64 than the launches of the
    same solve; errors over 24 matrices (at least 2400 entries of X, so their
    2-norm is known to 1.5%), 7% for the two samples."""
    p += pad
    err = {"1": [0.0, 0.0], "0": [0.0, 0.0]}
    for seed in range(24):
        gen = torch.Generator(device="cuda").manual_seed(seed)
        A = torch.randn((n, p), device="cuda", generator=gen).t()
        A64 = A.double()
        gamma = 0.03 * float(A64.norm(dim=0).max())
        top = torch.sort(A64.norm(dim=0), descending=True, stable=True)[1][:m]
        X0 = A64[:, top]
        if kind == "BL1":
            u, _, vt = torch.linalg.svd(X0, full_matrices=False)
            X, Z = _two_passes64(A64, u @ vt, gamma, True)
        else:
            X, Z = _two_passes64(A64, X0 / X0.norm(dim=0), gamma, False)
        for small in err:
            monkeypatch.setenv("GPSPCA_SMALL", small)
            if kind == "multi":
                r = gpu.solve_multistart(A, gpu.SL1, m, gamma, tol=0.0, max_iter=2)
            else:
                r = gpu.solve(A, gpu.SL1 if m == 1 else gpu.BL1, m, gamma, tol=0.0, max_iter=2)
            err[small][0] += float((r.X.double() - X).square().sum())
            err[small][1] += float((r.Z.double() - Z).square().sum())
    ratio = [(a / b) ** 0.5 for a, b in zip(err["1"], err["0"])]
    print(f"\n[accuracy] {kind}{m} p={p} n={n} X {ratio[0]:.3f} Z {ratio[1]:.3f}", flush=True)
    assert max(ratio) <= 1.07


@pytest.mark.parametrize("p,n,m", [(100, 1000, 1), (200, 2000, 5)])
def test_start_inside_an_output_survives_a_given_up_solve(gpu, p, n, m, monkeypatch):
    """X0 is read before anything is written, so it may lie in the buffer of an
    output.  A persistent solve that gives up (its barriers may not wait here) runs
    again from X0 and must not have written its outputs."""
    A = to_device(W.planted_block(p, n, 2, 3, k=30)[0])
    M = gpu.matrix(A)
    form, gamma, iters = (O.SL1 if m == 1 else O.BL1), 0.08 * float(A.norm(dim=0).max()), 6
    X0 = x_to_device(fp32_round(W.random_orthonormal(p, m, 4)))
    want = gpu.solve(A, form, m, gamma, X0=X0, tol=0.0, max_iter=iters)
    ws = torch.empty(gpu.workspace_bytes(A, form, m, iters) + 256, dtype=torch.uint8, device="cuda")
    ws = ws[(-ws.data_ptr()) % 256:]
    words = (n + 31) // 32
    for wait in ("0", None):
        monkeypatch.delenv("GPSPCA_SMALL_WAIT", raising=False)
        if wait is not None:
            monkeypatch.setenv("GPSPCA_SMALL_WAIT", wait)
        for place in range(2):
            X = torch.empty((m, p), device="cuda")
            Z = torch.empty((m, n), device="cuda")
            sup = torch.empty((m, words), dtype=torch.int32, device="cuda")
            at = (X, Z)[place].view(-1)[:m * p]
            at.copy_(X0.t().reshape(-1))
            nit = ctypes.c_int(0)
            trace = (ctypes.c_double * iters)()
            rc = gpu.load().gpspca_solve(ctypes.byref(M), form, m, gamma, None, at.data_ptr(), 0.0,
                                         iters, ws.data_ptr(), ws.numel(),
                                         torch.cuda.current_stream().cuda_stream, X.data_ptr(),
                                         Z.data_ptr(), sup.data_ptr(), trace, ctypes.byref(nit))
            assert rc == gpu.MAXITER and nit.value == iters
            np.testing.assert_allclose(list(trace), want.trace, rtol=1e-5)
            assert float((X.t() - want.X).norm() / want.X.norm()) <= 1e-5
            assert float((Z.t() - want.Z).norm() / want.Z.norm()) <= 1e-5


def _kernels(gpu, fn):
    """(result of fn, dominant kernel, its timed launches) by the library's timing."""
    gpu.profile_read()
    gpu.profile_enable(True)
    try:
        r = fn()
    finally:
        gpu.profile_enable(False)
    _, launches, name = gpu.profile_read()
    return r, name, launches


# (form, m, p, n, name as launches): solves of several workgroups, with one and with
# two barriers a pass
SMALL = [("SL1", 1, 100, 1000, "k_pass_m1"), ("SL1", 1, 400, 4000, "k_pass_m1"),
         ("BL1", 5, 200, 2000, "k_corr_mfma"), ("multi", 4, 100, 1000, "k_corr_mfma")]


@pytest.mark.parametrize("form,m,p,n,other", SMALL)
def test_small_solves_take_the_persistent_kernel(gpu, form, m, p, n, other, monkeypatch):
    """What ran, by the timing of launches, and with the timing on the same bits as
    without: one k_small; after a barrier's wait that ran out the passes as
    launches; k_small again with a longer limit; the launches alone when told so."""
    A = to_device(W.planted_block(p, n, 2, 3, k=30)[0])
    gamma, iters = 0.1 * float(A.norm(dim=0).max()), 7

    def solve():
        if form == "multi":
            return gpu.solve_multistart(A, gpu.SL1, m, gamma, tol=0.0, max_iter=iters)
        return gpu.solve(A, gpu.SL1 if m == 1 else gpu.BL1, m, gamma, tol=0.0, max_iter=iters)

    plain = solve()
    r, name, launches = _kernels(gpu, solve)
    assert (name, launches) == ("k_small", 1) and torch.equal(r.X, plain.X)
    monkeypatch.setenv("GPSPCA_SMALL_WAIT", "0")
    r, name, launches = _kernels(gpu, solve)
    assert (name, launches) == (other, 1 + iters)
    assert float((r.X - plain.X).norm() / plain.X.norm()) <= 1e-5
    r, name, launches = _kernels(gpu, solve)      # not tried again at once
    assert (name, launches) == (other, iters)
    monkeypatch.delenv("GPSPCA_SMALL_WAIT")
    r, name, launches = _kernels(gpu, solve)
    assert (name, launches) == ("k_small", 1) and torch.equal(r.X, plain.X)
    monkeypatch.setenv("GPSPCA_SMALL", "0")
    assert _kernels(gpu, solve)[1:] == (other, iters)


@pytest.mark.parametrize("form,m,p,n,other", SMALL)
def test_autotuning_a_small_matrix_does_not_slow_it(gpu, form, m, p, n, other):
    """Whole solves of these sizes are faster by the persistent kernel (1.1 to 2.4
    times), so it is what the autotuner has to choose, and later solves give the bits
    of untuned ones."""
    A = to_device(W.planted_block(p, n, 2, 3, k=30)[0])
    gamma = 0.1 * float(A.norm(dim=0).max())

    def solve():
        if form == "multi":
            return gpu.solve_multistart(A, gpu.SL1, m, gamma, tol=0.0, max_iter=7)
        return gpu.solve(A, gpu.SL1 if m == 1 else gpu.BL1, m, gamma, tol=0.0, max_iter=7)

    plain = solve()
    try:
        rep = gpu.autotune(A, gpu.BL1 if form == "BL1" else gpu.SL1, m, gamma, passes=20)
        print(f"\n[autotune] {form} m={m} {rep}", flush=True)
        assert rep["choice"].startswith("k_small")
        r, name, launches = _kernels(gpu, solve)
        assert (name, launches) == ("k_small", 1) and torch.equal(r.X, plain.X)
    finally:
        gpu.autotune_clear()


@pytest.mark.parametrize("pad", [0, 3], ids=["packed", "bytes"])
@pytest.mark.parametrize("to", [O.BF16, O.E4M3], ids=["bf16", "e4m3"])
@pytest.mark.parametrize("p", [1, 3, 5, 60, 63, 64, 65, 252, 255, 256, 257])
def test_quantize_short_columns(gpu, p, to, pad):
    """Codes and scales bit for bit around the shapes of the shortest columns, with
    columns past the last full workgroup and rows past p untouched."""
    n = 37
    A = W.gaussian(p, n, p)
    A[:, 1] = 0.0
    A[:, 2] *= 1e-39
    ldq = (p + 15) // 16 * 16 + pad
    es = 2 if to == O.BF16 else 1
    out = torch.full((n, ldq * es), 0x5A, dtype=torch.uint8, device="cuda")
    sc = torch.full((n,), -1.0, dtype=torch.float32, device="cuda")
    M = gpu.matrix(to_device(A, lda=p + pad))
    assert gpu.load().gpspca_quantize(ctypes.byref(M), int(to), out.data_ptr(), ldq, sc.data_ptr(),
                                      torch.cuda.current_stream().cuda_stream) == 0
    got = out.cpu().numpy()
    got = got.view(np.uint16) if es == 2 else got
    assert (got.view(np.uint8)[:, p * es:] == 0x5A).all()
    ref, ref_sc = O.quantize(A, to, ldq=ldq)
    np.testing.assert_array_equal(got[:, :p].T, ref[:p])
    np.testing.assert_array_equal(sc.cpu().numpy(), ref_sc if to == O.E4M3 else np.ones(n))


@pytest.mark.parametrize("p", [1, 4, 63, 255, 256, 257, 511, 512, 513, 1023, 1024, 1025])
def test_column_norms_of_short_columns(gpu, p):
    """FP64 norms of every storage type around the lengths where the kernel changes."""
    n = 133
    A = W.gaussian(p, n, 70 + p)
    ref = np.sqrt((A.astype(np.float64) ** 2).sum(axis=0))
    for lda in (p | 1, (p + 3) // 4 * 4 + 4):
        got = gpu.column_norms(to_device(A, lda=lda)).cpu().numpy()
        np.testing.assert_allclose(got, ref, rtol=1e-14, atol=0)
    for to in (O.BF16, O.E4M3):
        Aq, sc = gpu.quantize(to_device(A), torch.bfloat16 if to == O.BF16
                              else torch.float8_e4m3fn)
        codes, scale = O.quantize(A, to)
        deq = O.dequantize(codes, to, scale, p)
        got = gpu.column_norms(Aq, col_scale=sc).cpu().numpy()
        np.testing.assert_allclose(got, np.sqrt((deq ** 2).sum(axis=0)), rtol=1e-14, atol=0)


@pytest.mark.parametrize("store", ["f32", "odd", "bf16", "e4m3"])
@pytest.mark.parametrize("m", [2, 5, 16, 17, 32, 33, 64])
def test_forced_shared_x_kernel_is_the_one_that_runs(gpu, m, store, monkeypatch):
    """GPSPCA_CORR_KERNEL=sh gives k_corr_sh for every storage type, alignment and
    component group, except 8-bit codes with more than 32 components."""
    monkeypatch.setenv("GPSPCA_CORR_KERNEL", "sh")
    p, n = 203, 1500
    A, scale = to_device(W.gaussian(p, n, m), lda=203 if store == "odd" else 204), None
    if store in ("bf16", "e4m3"):
        A, scale = gpu.quantize(A, torch.bfloat16 if store == "bf16" else torch.float8_e4m3fn)
    _, name, launches = _kernels(gpu, lambda: gpu.solve(A, gpu.BL1, m, 0.5, tol=0.0, max_iter=3,
                                                        col_scale=scale))
    assert name == ("k_corr_qw" if store == "e4m3" and m > 32 else "k_corr_sh") and launches == 3


@pytest.mark.parametrize("m", [1, 2, 5, 8, 9, 16, 17, 32, 33, 48, 49, 64])
def test_start_projection_beyond_the_gram_matrix(gpu, m):
    """A start whose singular values fall to 1e-12 of the largest (to 1e-8 after its
    rounding to FP32, whose squares are the rounding of the Gram matrix): the call
    refuses it, or returns a finite X in which the direction of the largest value,
    resolved like in any other start, is that of the polar factor."""
    p, n = 200, 400
    rng = np.random.default_rng(m)
    U = np.linalg.qr(rng.standard_normal((p, m)))[0]
    V = np.linalg.qr(rng.standard_normal((m, m)))[0]
    sv = np.geomspace(1.0, 1e-12, m) if m > 1 else np.ones(1)
    X0 = fp32_round(3.0 * (U * sv) @ V.T)
    A = to_device(W.gaussian(p, n, 11))
    try:
        X = gpu.solve(A, gpu.BL1, m, 0.5, X0=x_to_device(X0), tol=0.0, max_iter=1).X
    except gpu.GpspcaError as e:
        assert m > 1 and e.code == gpu.EINVAL
        return
    X = X.double().cpu().numpy()
    u, _, vt = np.linalg.svd(X0, full_matrices=False)
    assert np.isfinite(X).all()
    np.testing.assert_allclose(X @ vt[0], u[:, 0], atol=1e-5)


@pytest.mark.parametrize("stream", [0, 1, 2], ids=["null", "legacy", "per_thread"])
def test_small_solve_on_the_default_streams(gpu, stream):
    """The NULL stream and the special handles of the default streams."""
    A = to_device(W.planted_block(100, 1000, 2, 3, k=30)[0])
    gamma = 0.1 * float(A.norm(dim=0).max())
    want = gpu.solve(A, gpu.SL1, 1, gamma, tol=0.0, max_iter=7)
    M = gpu.matrix(A)
    ws = torch.empty(gpu.workspace_bytes(A, gpu.SL1, 1, 7) + 256, dtype=torch.uint8, device="cuda")
    ws = ws[(-ws.data_ptr()) % 256:]
    X, Z = torch.empty((1, 100), device="cuda"), torch.empty((1, 1000), device="cuda")
    torch.cuda.synchronize()
    rc = gpu.load().gpspca_solve(ctypes.byref(M), gpu.SL1, 1, gamma, None, None, 0.0, 7,
                                 ws.data_ptr(), ws.numel(), stream, X.data_ptr(), Z.data_ptr(),
                                 None, None, None)
    assert rc == gpu.MAXITER
    torch.cuda.synchronize()
    assert torch.equal(X.t(), want.X) and torch.equal(Z.t(), want.Z)


@pytest.mark.parametrize("store", ["f32", "bf16"])
@pytest.mark.parametrize("form,m,p,n", [(O.SL0, 1, 100, 1000), (O.SL0, 1, 300, 3100),
                                        (O.BL0, 2, 120, 900), (O.BL0, 5, 200, 2000),
                                        (O.BL0, 8, 130, 1400)])
def test_small_solves_of_the_l0_forms(gpu, form, m, p, n, store):
    """Hard-threshold solves by the persistent kernel against the oracle, with gamma
    picked away from ties along the oracle's iterates."""
    iters = 6
    A = W.planted_block(p, n, min(m, 2), p + m, k=max(4, n // 25))[0]
    Ad, A64 = to_device(A, lda=p | 1), A.astype(np.float64)
    if store == "bf16":
        Ad, _ = gpu.quantize(to_device(A), torch.bfloat16)
        A64 = O.dequantize(O.quantize(A, O.BF16)[0], O.BF16, None, p)
    X0 = fp32_round(O.init(A64, m)[0])
    mu = None if m == 1 else list(np.linspace(1.0, 0.8, m))
    gamma = pick_gamma(A64, form, m, mu, X0, W.gamma_absolute(A64, True, 0.05), iters=iters)
    ref = O.solve(A64, form, m, gamma, mu=mu, X0=X0, tol=0.0, max_iter=iters)
    r, name, launches = _kernels(gpu, lambda: gpu.solve(
        Ad, int(form), m, gamma, mu=mu, X0=x_to_device(X0), tol=0.0, max_iter=iters))
    assert (name, launches) == ("k_small", 1)
    assert rel(r.X.cpu().numpy(), ref["X"]) <= 1e-5
    assert rel(r.Z.cpu().numpy(), ref["Z"]) <= 1e-5
    np.testing.assert_allclose(r.trace, ref["trace"], rtol=1e-5)
    np.testing.assert_array_equal(r.Z.cpu().numpy() != 0, ref["Z"] != 0)
