"""The scan where strips end and chunks begin by the fill of their rounds: 96 strips at
10 and 11 passes (FP64 and FP32), 192 at 16 and 17, 240 (a full round) at 24576 and
24577 of k.  Sampled entries against the oracle; the maximum of a sampled row and
column in its last element."""
import numpy as np
import pytest

from gpu_util import announce, dev, host
from oracle.ozaki2 import os_ii

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2602_02549_amd as oz  # noqa: E402


@pytest.mark.parametrize("m,k,dtype", [
    (1536, 5120, np.float64), (1530, 5121, np.float64), (3072, 2560, np.float32),
    (3070, 2561, np.float32), (3072, 8192, np.float64), (3071, 8193, np.float64),
    (3840, 24576, np.float64), (3833, 24577, np.float64)])
def test_strips(m, k, dtype):
    announce(f"scan strips m={m} k={k} {dtype.__name__}")
    n, N = 5, 6
    rng = np.random.default_rng(m + k)
    A = (rng.random((m, k)) - 0.5).astype(dtype)
    B = (rng.random((k, n)) - 0.5).astype(dtype)
    A[m - 1, k - 1] = B[k - 1, n - 1] = 100
    A[m // 2] = 0
    got = host(oz.gemm(dev(A), dev(B), N))
    rows, cols = np.array([0, m // 2, m - 1]), np.array([0, n - 1])
    assert np.array_equal(got[np.ix_(rows, cols)], os_ii(A, B, N, rows=rows, cols=cols))
