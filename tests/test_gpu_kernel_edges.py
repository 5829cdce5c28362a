"""Edges of the kernels' register and tile shapes: the smallest and largest
sizes of each variant, the remainders between them, odd leading dimensions."""
import ctypes

import numpy as np
import pytest
import torch

import oracle as O
from workloads import generators as W

from _util import TD, to_device

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
