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
