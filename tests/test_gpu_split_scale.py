"""The scaling product split for two workgroups per CU (more than 32 tiles, 256 groups
of k or more), at the edges of that rule: the maxima of Cbar and every stage after
them as without a split, and sampled entries as the oracle."""
import numpy as np
import pytest

from gpu_util import announce, dev, host
from oracle.ozaki2 import os_ii

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2602_02549_amd as oz  # noqa: E402


# 54 tiles of 255 groups (one per CU) and of 256; 100 and 33 tiles; 32 (one per CU)
@pytest.mark.parametrize("m,n,k", [(1100, 700, 32640), (1100, 700, 32641), (1270, 1153, 33000),
                                   (1300, 300, 66000), (1000, 500, 66000)])
def test_two_per_cu(m, n, k):
    announce(f"split scaling product {m}x{n}x{k}")
    N = 2
    rng = np.random.default_rng(m + n + k)
    A, B = rng.random((m, k)) - 0.5, rng.random((k, n)) - 0.5
    A[m - 1, k - 1] = B[k - 1, n - 1] = 100.0
    dA, dB = dev(A), dev(B)
    got = {kk: host(v) for kk, v in oz.debug_stages(dA, dB, N, crt_stages=False).items()
           if kk in ("rmax", "cmax", "mu", "nu", "CT")}
    rc, prev = oz.ozaki2_debug_tuning(oz.KNOB_SPLIT_K, 1)
    assert rc == oz.OK
    try:
        want = oz.debug_stages(dA, dB, N, crt_stages=False)
        for kk, v in got.items():
            assert np.array_equal(v, host(want[kk])), kk
    finally:
        oz.ozaki2_debug_tuning(oz.KNOB_SPLIT_K, prev)
    rows, cols = np.array([0, m // 2, m - 1]), np.array([0, n // 2, n - 1])
    assert np.array_equal(got["CT"].T[np.ix_(rows, cols)], os_ii(A, B, N, rows=rows, cols=cols))
