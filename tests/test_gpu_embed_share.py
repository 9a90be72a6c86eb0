"""The embedding's residues with more tiles than workgroups and very uneven sides (the
share of each side depends on the tiles and on N): sampled entries against the oracle,
one, two and three limbs and exact steps."""
import numpy as np
import pytest

from gpu_util import announce, dev, host
from oracle.complex_gemm import os_ii_complex
from workload import complex_gemm_inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2602_02549_amd as oz  # noqa: E402


@pytest.mark.parametrize("N", [2, 15, 24, 33])
@pytest.mark.parametrize("m,n,k", [(9000, 3, 700), (3, 9000, 700)])
def test_share(m, n, k, N):
    announce(f"embedding share {m}x{n}x{k} N={N}")
    A, B = complex_gemm_inputs(m, n, k, phi=1.0, seed=m + N)
    rows, cols = np.array([0, m // 2, m - 1]), np.array([0, n // 2, n - 1])
    got = host(oz.zgemm(dev(A), dev(B), N))
    assert np.array_equal(got[np.ix_(rows, cols)], os_ii_complex(A, B, N, rows=rows, cols=cols))
