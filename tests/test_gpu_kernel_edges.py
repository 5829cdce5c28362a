"""Edges of the kernels' register and tile shapes: the smallest and largest
sizes of each variant, the remainders between them, odd leading dimensions."""
import ctypes

import numpy as np
import pytest
import torch

import oracle as O
from workloads import generators as W

from _util import (TD, corr_band, fp32_round, rel, tie_mask, to_device, x_to_device)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("pad", [0, 3], ids=["packed", "bytes"])
@pytest.mark.parametrize("to", [O.BF16, O.E4M3], ids=["bf16", "e4m3"])
@pytest.mark.parametrize("p", [1, 3, 4, 255, 1024, 1025, 2560, 2563, 10240, 10241, 20480, 20483,
                               40960, 40961])
def test_quantize_column_lengths(gpu, p, to, pad):
    """Codes and scales bit for bit at the first and last length of every
    register shape, with and without packed stores; rows past p untouched."""
    n = 7
    A = W.gaussian(p, n, p)
    A[:, 1] = 0.0
    A[:, 2] *= 1e-39
    A[0, 3] = np.inf
    ldq = (p + 15) // 16 * 16 + pad
    lda = p + pad
    Ad = to_device(A, lda=lda)
    es = 2 if to == O.BF16 else 1
    out = torch.full((n, ldq * es), 0x5A, dtype=torch.uint8, device="cuda")
    sc = torch.full((n,), -1.0, dtype=torch.float32, device="cuda")
    M = gpu.matrix(Ad)
    rc = gpu.load().gpspca_quantize(ctypes.byref(M), int(to), out.data_ptr(), ldq, sc.data_ptr(),
                                    torch.cuda.current_stream().cuda_stream)
    assert rc == 0
    got = out.cpu().numpy()
    got = got.view(np.uint16) if es == 2 else got
    assert (got.view(np.uint8)[:, p * es:] == 0x5A).all()
    keep = [c for c in range(n) if c != 3]
    ref, ref_sc = O.quantize(A[:, keep], to, ldq=ldq)
    np.testing.assert_array_equal(got[keep, :p].T, ref[:p])
    if to == O.E4M3:
        np.testing.assert_array_equal(sc.cpu().numpy()[keep], ref_sc)
        # an infinite entry: inf / inf saturates like a NaN, the others vanish
        assert np.isinf(sc[3].item()) and got[3, 0] & 0x7F == 0x7E
        assert not (got[3, 1:p] & 0x7F).any()
    else:
        assert (sc == 1.0).all() and got[3, 0] == 0x7F80


@pytest.mark.parametrize("p", [1, 3, 5, 15, 17, 63, 255, 257, 1023, 1025, 4100])
def test_column_norms_lengths(gpu, p):
    """FP64 norms of every storage type around the 16-byte segments, their
    64-lane rows and the 4-segment batches; an odd leading dimension in FP32."""
    n = 133
    A = W.gaussian(p, n, 50 + p)
    A[:, 3] = 0.0
    ref = np.sqrt((A.astype(np.float64) ** 2).sum(axis=0))
    for lda in (p, (p + 3) // 4 * 4 + 4):
        got = gpu.column_norms(to_device(A, lda=lda)).cpu().numpy()
        np.testing.assert_allclose(got, ref, rtol=1e-14, atol=0)
    for to in (O.BF16, O.E4M3):
        Aq, sc = gpu.quantize(to_device(A), TD[to])
        codes, scale = O.quantize(A, to)
        deq = O.dequantize(codes, to, scale, p)
        got = gpu.column_norms(Aq, col_scale=sc).cpu().numpy()
        np.testing.assert_allclose(got, np.sqrt((deq ** 2).sum(axis=0)), rtol=1e-14, atol=0)


# (p, n, m): fewer rows than one stage or slot, one row past a stage, fewer tiles
# than waves, one tile past a round of 32, ragged tiles, every component group
SH_SHAPES = [(3, 40, 2), (17, 16, 16), (63, 700, 5), (65, 130, 17), (128, 4099, 33),
             (257, 8193 * 16 + 1, 8), (1003, 3001, 32), (1025, 2000, 64)]


@pytest.mark.parametrize("store", ["f32", "odd", "bf16", "e4m3"])
@pytest.mark.parametrize("p,n,m", SH_SHAPES)
def test_shared_x_correlation(gpu, p, n, m, store, monkeypatch):
    """One pass of k_corr_sh in every mode and component group against FP64."""
    if m > p:
        m = p
    print(f"\n[corr sh] {store} p={p} n={n} m={m}", flush=True)
    monkeypatch.setenv("GPSPCA_CORR_KERNEL", "sh")
    A = W.gaussian(p, n, p + m)
    scale = None
    if store in ("f32", "odd"):
        Ad = to_device(A, lda=(p + 3) // 4 * 4 if store == "f32" else p | 1)
        A64 = A.astype(np.float64)
    else:
        to = O.BF16 if store == "bf16" else O.E4M3
        Ad, scale = gpu.quantize(to_device(A), TD[to])
        A64 = O.dequantize(*((c := O.quantize(A, to))[0], to, c[1], p))
    X = fp32_round(W.random_orthonormal(p, m, 7))
    gamma, mu = 0.9, np.linspace(1.0, 0.7, m)
    out = gpu.step(Ad, O.BL1, x_to_device(X), gamma, mu=list(mu), col_scale=scale)
    ref = O.step(A64, O.BL1, X, gamma, mu=mu)
    S = out.S.cpu().numpy().astype(np.float64)
    ties = tie_mask(A64, X, O.BL1, gamma, mu)
    np.testing.assert_array_equal((S != 0)[~ties], (ref["S"] != 0)[~ties])
    assert np.all(np.abs(S - ref["S"]) <= corr_band(A64, X) * mu[None, :] + 1e-7 * np.abs(ref["S"]))
    assert rel(out.G.cpu().numpy(), ref["G"]) <= 1e-5
    np.testing.assert_allclose(out.f, ref["f"], rtol=1e-5)


@pytest.mark.parametrize("store", ["f32", "odd", "bf16"])
def test_shared_x_correlation_non_finite(gpu, store, monkeypatch):
    """An infinity or an entry near the FP32 limit keeps the meaning it has in
    plain FP32 products (the split parts of both are NaN); a NaN marks no entry."""
    monkeypatch.setenv("GPSPCA_CORR_KERNEL", "sh")
    p, n, m = 261, 200, 40
    A = W.gaussian(p, n, 5)
    # bfloat16's largest finite value is 3.39e38; 3.4e38 would round to infinity
    A[7, 3], A[8, 4], A[9, 5] = np.inf, 3.38e38 if store == "bf16" else 3.4e38, np.nan
    Ad = to_device(A, lda=264 if store == "f32" else 261)
    if store == "bf16":
        Ad, _ = gpu.quantize(to_device(A), torch.bfloat16)
        A = Ad.t().contiguous().float().cpu().numpy().T
    X = fp32_round(W.random_orthonormal(p, m, 8))
    with pytest.raises(gpu.GpspcaError):
        gpu.step(Ad, O.BL1, x_to_device(X), 0.5)
    keep = [c for c in range(n) if c != 3]
    B = np.ascontiguousarray(A[:, keep])
    Bd = to_device(B, lda=264 if store == "f32" else 261)
    if store == "bf16":
        Bd, _ = gpu.quantize(Bd, torch.bfloat16)
    S = gpu.step(Bd, O.BL1, x_to_device(X * 2.0 ** -20), 0.5).S.cpu().numpy()
    big = keep.index(4)
    want = B[:, big].astype(np.float64) @ (X * 2.0 ** -20)
    np.testing.assert_allclose(S[big], np.sign(want) * np.maximum(np.abs(want) - 0.5, 0), rtol=1e-6)
    assert not S[keep.index(5)].any()


def test_noalloc_limit_of_unaligned_columns(gpu, monkeypatch):
    """The largest problem that fits the library's scratch with the vector-ALU
    correlation still fits when the default kernel needs more."""
    p, m = 101, 8
    hi = 1_600_000
    buf = torch.randn((hi, p), device="cuda")

    def fits(n):
        try:
            gpu.solve_noalloc(buf[:n].t(), gpu.BL1, m, 1e3, tol=0.0, max_iter=1)
            return True
        except gpu.GpspcaError as e:
            assert e.code == gpu.ENOMEM
            return False

    monkeypatch.setenv("GPSPCA_CORR_KERNEL", "valu")
    lo = 1_000_000
    assert fits(lo) and not fits(hi)
    while hi - lo > 1:
        mid = (lo + hi) // 2
        lo, hi = (mid, hi) if fits(mid) else (lo, mid)
    monkeypatch.delenv("GPSPCA_CORR_KERNEL")
    assert fits(lo)


def _small_case(gpu, kind, Ad, scale, A64, m, iters):
    """(GPU call, oracle results per problem) of one persistent solve."""
    top = np.sqrt((A64 ** 2).sum(axis=0)).max()
    if kind in ("path", "multi"):
        form = O.SL1
        order = np.argsort(-(A64 ** 2).sum(axis=0), kind="stable")
        gams = [0.1 * top * (1 + 0.4 * (j if kind == "path" else 0)) for j in range(m)]
        starts = [order[0 if kind == "path" else j] for j in range(m)]
        refs = [O.solve(A64, form, 1, gams[j],
                        X0=(A64[:, starts[j]] / np.linalg.norm(A64[:, starts[j]]))[:, None],
                        tol=0.0, max_iter=iters) for j in range(m)]
        if kind == "path":
            return (lambda: gpu.solve_path(Ad, form, gams, tol=0.0, max_iter=iters, col_scale=scale),
                    refs)
        return (lambda: gpu.solve_multistart(Ad, form, m, gams[0], tol=0.0, max_iter=iters,
                                             col_scale=scale), refs)
    form = {"SL1": O.SL1, "BL1": O.BL1, "BL1X": O.BL1X}[kind]
    gamma = 0.1 * top
    X0 = O.init(A64, m)[0]
    ref = O.solve(A64, form, m, gamma, X0=X0, tol=0.0, max_iter=iters)
    return (lambda: gpu.solve(Ad, int(form), m, gamma, tol=0.0, max_iter=iters, col_scale=scale),
            [ref])


# (p, n): one row, fewer columns than a tile, one workgroup, one tile past the
# workgroups' shares, ragged quads, rows past the threads' quads, the LDS limit
@pytest.mark.parametrize("store", ["f32", "bf16", "e4m3"])
@pytest.mark.parametrize("kind,m", [("SL1", 1), ("BL1", 5), ("BL1", 8), ("BL1X", 2), ("path", 6),
                                    ("multi", 16)])
@pytest.mark.parametrize("p,n", [(9, 15), (17, 129), (63, 1041), (101, 1003), (258, 2100),
                                 (2100, 300)])
def test_small_persistent_solve(gpu, p, n, kind, m, store, monkeypatch):
    """Solves that run as one persistent kernel (and those just past its limits)
    against the oracle, twice bitwise the same, and in pieces of one launch."""
    m = min(m, p, n)
    iters = 7
    print(f"\n[small] {kind} {store} p={p} n={n} m={m}", flush=True)
    A = W.planted_block(p, n, 2, p + n, k=max(2, n // 20))[0]
    scale = None
    if store == "f32":
        Ad, A64 = to_device(A, lda=p | 1), A.astype(np.float64)
    else:
        to = O.BF16 if store == "bf16" else O.E4M3
        Ad, scale = gpu.quantize(to_device(A), TD[to])
        codes, sc = O.quantize(A, to)
        A64 = O.dequantize(codes, to, sc, p)
    fn, refs = _small_case(gpu, kind, Ad, scale, A64, m, iters)
    a, b = fn(), fn()
    assert torch.equal(a.X, b.X) and torch.equal(a.Z, b.Z) and torch.equal(a.support, b.support)
    if len(refs) == 1 and kind not in ("path", "multi"):
        assert rel(a.X.cpu().numpy(), refs[0]["X"]) <= 1e-5
        np.testing.assert_allclose(a.trace, refs[0]["trace"], rtol=1e-5)
        assert a.n_iter == refs[0]["n_iter"]
    else:
        for j, ref in enumerate(refs):
            assert rel(a.X[:, j].cpu().numpy(), ref["X"][:, 0]) <= 1e-5
            np.testing.assert_allclose(a.traces[j], ref["trace"], rtol=1e-5)
    # a barrier that never waits long enough: the passes run as separate launches
    monkeypatch.setenv("GPSPCA_SMALL_WAIT", "0")
    c = fn()
    assert rel(c.X.cpu().numpy(), a.X.cpu().numpy()) <= 1e-5 and c.n_iter == a.n_iter


def test_small_solve_of_many_passes_and_threads(gpu):
    """More passes than one launch holds, stopped by the tolerance or not, from
    several threads on their own streams at once: bitwise the solo results."""
    import threading
    A = to_device(W.planted_block(150, 1500, 2, 3, k=40)[0])
    top = float(A.norm(dim=0).max())
    jobs = [(g, f, m, tol) for g in (0.05, 0.12) for f, m in ((gpu.SL1, 1), (gpu.BL1, 4))
            for tol in (0.0, 1e-9)]

    def run(job):
        g, f, m, tol = job
        return gpu.solve(A, f, m, g * top, tol=tol, max_iter=600)

    solo = [run(j) for j in jobs]
    assert any(r.n_iter == 600 for r in solo)
    got = [None] * len(jobs)

    def work(i):
        with torch.cuda.stream(torch.cuda.Stream()):
            got[i] = run(jobs[i])

    torch.cuda.synchronize()
    ts = [threading.Thread(target=work, args=(i,)) for i in range(len(jobs))]
    [t.start() for t in ts]
    [t.join() for t in ts]
    for a, b in zip(solo, got):
        assert torch.equal(a.X, b.X) and torch.equal(a.Z, b.Z) and a.trace == b.trace


@pytest.mark.parametrize("kappa", [1.0, 30.0, 3e3, 1e7, 1e12])
@pytest.mark.parametrize("m", [1, 2, 5, 8, 9, 16, 17, 32, 33, 48, 49, 64])
def test_start_projection_by_size_and_condition(gpu, m, kappa):
    """The polar factor of a start whose Gram matrix has condition kappa^2, in
    every size of the Newton iteration and beyond its reach (Jacobi).  The X_0 of a
    one-pass solve against numpy's SVD; FP64 throughout, so up to the rounding of
    the FP32 start and result and its amplification by kappa."""
    p, n = 200, 400
    rng = np.random.default_rng(m)
    U = np.linalg.qr(rng.standard_normal((p, m)))[0]
    V = np.linalg.qr(rng.standard_normal((m, m)))[0]
    sv = np.geomspace(1.0, 1.0 / kappa, m) if m > 1 else np.ones(1)
    X0 = fp32_round(3.0 * (U * sv) @ V.T)
    u, _, vt = np.linalg.svd(X0, full_matrices=False)
    A = W.gaussian(p, n, 11)
    try:
        res = gpu.solve(to_device(A), gpu.BL1, m, 0.5, X0=x_to_device(X0), tol=0.0, max_iter=1)
    except gpu.GpspcaError as e:
        # the Gram matrix's smallest eigenvalues are FP64 rounding here
        assert kappa == 1e12 and e.code == gpu.EINVAL
        return
    # the FP64 Gram matrix resolves singular values down to 1e-8 of the largest
    tol = 1e-6 if kappa <= 3e3 else 1e-2
    if kappa <= 1e7:
        assert rel(res.X.cpu().numpy(), u @ vt) <= tol
    X = res.X.double().cpu().numpy()
    if kappa <= 3e3:
        assert np.abs(X.T @ X - np.eye(m)).max() <= 1e-6


@pytest.mark.parametrize("m,mu", [(5, "graded"), (8, "one"), (12, "graded"), (24, "one"),
                                  (33, "one"), (64, "one")])
def test_block_retraction_sizes(gpu, m, mu):
    """Block solves of every retraction size, plain and with graded weights
    (whose Gram matrix has a condition number of m^4 or more)."""
    p, n, iters = 300, 1500, 5
    A32 = W.planted_block(p, n, min(m, 8), 60 + m, k=20)[0]
    A64 = A32.astype(np.float64)
    w = np.ones(m) if mu == "one" else 1.0 / np.sqrt(np.arange(1, m + 1))
    X0 = fp32_round(O.init(A64, m)[0])
    gamma = W.gamma_absolute(A64, False, 0.05)
    ref = O.solve(A64, O.BL1, m, gamma, mu=w, X0=X0, tol=0.0, max_iter=iters)
    res = gpu.solve(to_device(A32), gpu.BL1, m, gamma, mu=list(w), X0=x_to_device(X0), tol=0.0,
                    max_iter=iters)
    assert rel(res.X.cpu().numpy(), ref["X"]) <= 1e-5
    np.testing.assert_allclose(res.trace, ref["trace"], rtol=1e-5)


@pytest.mark.parametrize("order", ["ties", "falling", "rising", "equal"])
@pytest.mark.parametrize("n,m", [(1, 1), (63, 63), (64, 64), (257, 5), (1024, 16), (1025, 64),
                                 (20011, 16), (100003, 64), (524288, 3), (600001, 64)])
def test_start_columns_selection(gpu, n, m, order):
    """The m starts of a one-pass multistart are the columns of largest norm, ties to
    the lower index, around the lanes, waves, workgroups and register range of the
    selection.  Column i is its index in signs, times a level: norms are exact
    whole numbers, and the signs of X_0 give the index back."""
    bits = 20
    i = np.arange(n)
    level = {"ties": np.random.default_rng(n + m).integers(1, 40, n), "falling": n - i,
             "rising": i + 1, "equal": np.full(n, 3)}[order].astype(np.float32)
    A = (2.0 * ((i[None, :] >> np.arange(bits)[:, None]) & 1) - 1.0).astype(np.float32) * level
    res = gpu.solve_multistart(to_device(A), gpu.SL1, m, 0.01, tol=0.0, max_iter=1)
    got = ((res.X.cpu().numpy() > 0) * (1 << np.arange(bits))[:, None]).sum(axis=0)
    np.testing.assert_array_equal(got, np.argsort(-level.astype(np.float64), kind="stable")[:m])


@pytest.mark.parametrize("p,n,m", [(17, 200, 2), (65, 1500, 4), (79, 600, 9), (129, 3000, 16),
                                   (16384, 150, 5), (16385, 150, 5), (16400, 150, 12),
                                   (200, 2000, 17), (113, 700, 64), (33000, 130, 20)])
@pytest.mark.parametrize("path", [False, True], ids=["block", "path"])
def test_gram_row_blocks(gpu, p, n, m, path, monkeypatch):
    """The Gram products of a pass by row blocks: remainders of 64 rows and of 16,
    both slicings of the partial sums, one to four component tiles; the diagonal
    alone on a gamma path.  Rounding of FP32 operands, as in the block solves above."""
    monkeypatch.setenv("GPSPCA_SMALL", "0")
    A32 = W.planted_block(p, n, min(m, 8), 90 + m, k=20)[0]
    A64 = A32.astype(np.float64)
    X0 = fp32_round(O.init(A64, m)[0])
    gamma = W.gamma_absolute(A64, False, 0.05)
    if path:
        g = [gamma * (1.0 + 0.01 * j) for j in range(m)]
        res = gpu.solve_path(to_device(A32), gpu.SL1, g, X0=x_to_device(X0), tol=0.0, max_iter=3)
        X = res.X.cpu().numpy()
        for j in range(m):
            ref = O.solve(A64, O.SL1, 1, g[j], X0=X0[:, [j]], tol=0.0, max_iter=3)
            assert rel(X[:, [j]], ref["X"]) <= 1e-5
    else:
        ref = O.solve(A64, O.BL1, m, gamma, X0=X0, tol=0.0, max_iter=3)
        res = gpu.solve(to_device(A32), gpu.BL1, m, gamma, X0=x_to_device(X0), tol=0.0, max_iter=3)
        assert rel(res.X.cpu().numpy(), ref["X"]) <= 1e-5
        np.testing.assert_allclose(res.trace, ref["trace"], rtol=1e-5)


@pytest.mark.parametrize("store", ["f32", "bf16", "e4m3"])
@pytest.mark.parametrize("active", ["one", "few", "clustered", "all"])
@pytest.mark.parametrize("p,n,m", [(64, 2_200_000, 5), (1028, 4097, 9), (1023, 5000, 16),
                                   (1000, 3000, 17), (2052, 700, 33), (67, 131, 64)])
def test_matrix_core_back_projection(gpu, p, n, m, active, store, monkeypatch):
    """G of one pass over lists of active columns: a single one, every 97th, the
    last ranges only, all (2148 columns a range at n = 2.2e6, more than one list);
    ragged rows; one to four component groups.  The same S in FP64 on the same
    stored values, so only the FP32 sums over a range differ."""
    monkeypatch.setenv("GPSPCA_BACKPROJ", "dense")
    m = min(m, p)
    gen = torch.Generator(device="cuda").manual_seed(p + n)
    ld = (p + 3) // 4 * 4
    buf = torch.randn((n, ld), device="cuda", generator=gen)
    i = torch.arange(n, device="cuda")
    on = {"one": i == n // 3, "few": i % 97 == 5, "clustered": i >= n - n // 9,
          "all": i >= 0}[active]
    buf *= on[:, None]
    A = buf[:, :p].t()
    scale, Av = None, A.double()
    if store != "f32":
        A, scale = gpu.quantize(A, TD[O.BF16 if store == "bf16" else O.E4M3])
        Av = A[:p].double() * (1.0 if scale is None else scale.double()[None, :])
    X = x_to_device(fp32_round(W.random_orthonormal(p, m, 7)))
    mu = np.linspace(1.0, 0.7, m)
    out = gpu.step(A, O.BL1, X, 0.05, mu=list(mu), col_scale=scale)
    ref = Av @ (out.S.double() * torch.tensor(mu, device="cuda"))
    assert (out.S != 0).any() and not (out.S[~on] != 0).any()
    assert rel(out.G.cpu().numpy(), ref.cpu().numpy()) <= 1e-5
