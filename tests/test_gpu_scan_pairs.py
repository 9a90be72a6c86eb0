"""The chunked scan of FP32 pairs, whose columns always go in chunks: one and many
columns, at, past and well past a chunk of 8192, against the oracle."""
import numpy as np
import pytest

from gpu_util import announce, dev, host
from oracle.complex_gemm import os_ii_complex, os_ii_complex_3m
from workload import complex_gemm_inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2602_02549_amd as oz  # noqa: E402


@pytest.mark.parametrize("form,oracle", [("4m", os_ii_complex), ("3m", os_ii_complex_3m)])
@pytest.mark.parametrize("m,n,k", [(20, 101, 8192), (20, 101, 8193), (5, 700, 4099), (70, 130, 20001)])
def test_pairs(form, oracle, m, n, k):
    announce(f"scan pairs {form} {m}x{n}x{k}")
    N = 5
    A, B = complex_gemm_inputs(m, n, k, phi=1.0, seed=m + n + k)
    A, B = A.astype(np.complex64), B.astype(np.complex64)
    B[k - 1, n - 1] *= 64          # the maximum of a column in its last element
    B[:, n // 2] = 0
    rows, cols = np.array([0, m // 2, m - 1]), np.array([0, n // 2, n - 1])
    got = host(oz.zgemm(dev(A), dev(B), N, form=form))
    assert np.array_equal(got[np.ix_(rows, cols)], oracle(A, B, N, rows=rows, cols=cols))
