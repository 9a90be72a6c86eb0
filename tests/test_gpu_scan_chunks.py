"""The chunked scan (few strips of A over a long k) at the edges of its chunks:
64, 128 and 256 rows per chunk, columns by the workgroup and in chunks (to 100
columns), k at and past a chunk; and columns of A so far apart that a strip's
32-bit offsets just reach and no longer reach them.  Every stage bit-exact
against the oracle."""
import numpy as np
import pytest

from gpu_util import announce, compare_stages, dev, host
from oracle.complex_gemm import os_ii_complex, os_ii_complex_3m
from oracle.ozaki2 import os_ii
from workload import complex_gemm_inputs, gemm_inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2602_02549_amd as oz  # noqa: E402


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("m,n,k", [
    (1, 1, 8193), (64, 100, 8192), (65, 101, 4097), (129, 3, 4097), (257, 99, 5000), (128, 2, 16385),
])
def test_chunk_stages(m, n, k, dtype):
    announce(f"scan chunks {m}x{n}x{k} {np.dtype(dtype).name}")
    N = 3
    A, B = gemm_inputs(m, n, k, phi=1.0, seed=m + n + k, dtype=dtype)
    A[m // 2] = 0.0
    B[:, n // 2] = 0.0
    B[k - 1, 0] *= 64          # the last element of a column and of a row count
    A[0, k - 1] *= 64
    got = {kk: host(v) for kk, v in oz.debug_stages(dev(A), dev(B), N, crt_stages=False).items()}
    C_ref, st = os_ii(A, B, N, stages=True)
    assert compare_stages(got, st, C_ref, N) == []


@pytest.mark.parametrize("form", ["4m", "3m"])
@pytest.mark.parametrize("m,n,k", [(33, 100, 4100), (70, 101, 8200)])
def test_chunks_complex(form, m, n, k):
    announce(f"scan chunks {form} {m}x{n}x{k}")
    N = 6
    A, B = complex_gemm_inputs(m, n, k, phi=1.0, seed=m + n)
    A[m - 1, k - 1] *= 64
    B[k - 1, n - 1] *= 64
    rows, cols = np.array([0, m // 2, m - 1]), np.array([0, n // 2, n - 1])
    want = (os_ii_complex_3m if form == "3m" else os_ii_complex)(A, B, N, rows=rows, cols=cols)
    got = host(oz.zgemm(dev(A), dev(B), N, form=form))
    assert np.array_equal(got[np.ix_(rows, cols)], want)


# 300 columns of doubles: offsets end just below 2^32, and past it
@pytest.mark.parametrize("lda", [1_780_000, 1_790_000])
def test_wide_pitch(lda):
    m, n, k, N = 40, 20, 300, 5
    announce(f"lda {lda}")
    A, B = gemm_inputs(m, n, k, phi=1.0, seed=lda)
    far = torch.empty((k, lda), dtype=torch.float64, device="cuda:0")
    far[:, :m] = dev(A.T)
    dB = dev(B.T)
    C = torch.zeros((n, m), dtype=torch.float64, device="cuda:0")
    rc = oz.ozaki2_gemm(m, n, k, far.data_ptr(), lda, dB.data_ptr(), k, C.data_ptr(), m, N)
    assert rc == oz.OK
    assert np.array_equal(host(C).T, os_ii(A, B, N))
    assert oz.ozaki2_sync_status() == oz.OK
