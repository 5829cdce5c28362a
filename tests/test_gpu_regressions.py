"""Faults that were found in the kernels and their dispatch, one test each."""
import numpy as np
import pytest
import torch

import oracle as O
from workloads import generators as W

from _util import fp32_round, to_device, x_to_device

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
    by 1.6e-6; totals every 32 rows leave the rounding of p / 32 additions,
    0.3 sqrt(313) 2^-24 = 3.2e-7, and that of a step's own products."""
    p, n, m = 10000, 6000, 64
    gen = torch.Generator(device="cuda").manual_seed(4)
    A = torch.randn((n, p), device="cuda", generator=gen).t()
    X = x_to_device(fp32_round(W.random_orthonormal(p, m, 9)))
    monkeypatch.setenv("GPSPCA_CORR_KERNEL", "sh")
    assert _correlation_error(gpu, A, X, A.t().double() @ X.double()) <= 5e-7
