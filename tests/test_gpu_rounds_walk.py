"""The walk in rounds where its pieces meet: a last round of two parts, of a tile each
(uncut) after a whole round, two whole rounds before a cut one, more tile rows than a
group of 16, and products reduced every 2^17 of k.  The same bits as with 128 x 128
tiles, which are not walked so, and as the oracle on sampled entries.  256 x 256 tiles
a slice: 16 (N = 22: 352 in all, 25: 400, 33: 528), 17 x 1 (N = 16: 272)."""
import numpy as np
import pytest

from gpu_util import announce, dev, host
from oracle.ozaki2 import os_ii

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2602_02549_amd as oz  # noqa: E402


@pytest.mark.parametrize("m,n,k,Ns", [(1024, 1000, 49300, (22, 25, 33)), (4352, 200, 33000, (16,)),
                                      (1024, 1000, 131200, (17,))])
def test_rounds_walk(m, n, k, Ns):
    rng = np.random.default_rng(m + n + k)
    A, B = rng.random((m, k)) - 0.5, rng.random((k, n)) - 0.5
    dA, dB = dev(A), dev(B)
    rows, cols = np.array([0, m // 2, m - 1]), np.array([0, n // 2, n - 1])
    for N in Ns:
        announce(f"rounds walk {m}x{n}x{k} N={N}")
        got = host(oz.gemm(dA, dB, N))
        rc, prev = oz.ozaki2_debug_tuning(oz.KNOB_GEMM_TILE, 2)
        assert rc == oz.OK
        try:
            assert np.array_equal(got, host(oz.gemm(dA, dB, N)))
        finally:
            oz.ozaki2_debug_tuning(oz.KNOB_GEMM_TILE, prev)
        assert np.array_equal(got[np.ix_(rows, cols)], os_ii(A, B, N, rows=rows, cols=cols))
