"""Split residue products at the edges of the rule for one workgroup per CU: 4 and 6
tiles a slice, 16 tiles below and at 2^17 of k, 25 at 2^17.  The same bits as without a
split, sampled entries as the oracle."""
import numpy as np
import pytest

from gpu_util import announce, dev, host
from oracle.ozaki2 import os_ii

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2602_02549_amd as oz  # noqa: E402


@pytest.mark.parametrize("m,n,k,N", [(250, 200, 9000, 16), (300, 250, 9000, 14), (500, 400, 9000, 8),
                                     (500, 400, 130945, 8), (620, 600, 130945, 5)])
def test_fill(m, n, k, N):
    announce(f"split fill {m}x{n}x{k} N={N}")
    rng = np.random.default_rng(m + n + k)
    A, B = rng.random((m, k)) - 0.5, rng.random((k, n)) - 0.5
    dA, dB = dev(A), dev(B)
    got = host(oz.gemm(dA, dB, N))
    rc, prev = oz.ozaki2_debug_tuning(oz.KNOB_SPLIT_K, 1)
    assert rc == oz.OK
    try:
        assert np.array_equal(got, host(oz.gemm(dA, dB, N)))
    finally:
        oz.ozaki2_debug_tuning(oz.KNOB_SPLIT_K, prev)
    rows, cols = np.array([0, m // 2, m - 1]), np.array([0, n // 2, n - 1])
    assert np.array_equal(got[np.ix_(rows, cols)], os_ii(A, B, N, rows=rows, cols=cols))
