"""Residue products whose tiles are walked in rounds over all XCDs (operands of
more than 96 MB a slice): the same bits as with 128 x 128 tiles, which are not,
and as the oracle on sampled entries.  16 tiles of 256 x 256 a slice with a last
round in parts, and 25 a slice, whose rounds end inside a group of tile rows."""
import numpy as np
import pytest

from gpu_util import announce, dev, host
from oracle.ozaki2 import os_ii

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2602_02549_amd as oz  # noqa: E402


@pytest.mark.parametrize("m,n,k,N", [(1024, 1000, 49300, 17), (1200, 1100, 39500, 12)])
def test_rounds(m, n, k, N):
    announce(f"rounds {m}x{n}x{k} N={N}")
    rng = np.random.default_rng(m + n + k)
    A = rng.random((m, k)) - 0.5
    B = rng.random((k, n)) - 0.5
    dA, dB = dev(A), dev(B)
    got = host(oz.gemm(dA, dB, N))
    rc, prev = oz.ozaki2_debug_tuning(oz.KNOB_GEMM_TILE, 2)
    assert rc == oz.OK
    try:
        assert np.array_equal(got, host(oz.gemm(dA, dB, N)))
    finally:
        oz.ozaki2_debug_tuning(oz.KNOB_GEMM_TILE, prev)
    rows, cols = np.array([0, m // 2, m - 1]), np.array([0, n // 2, n - 1])
    assert np.array_equal(got[np.ix_(rows, cols)], os_ii(A, B, N, rows=rows, cols=cols))
