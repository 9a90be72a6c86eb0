"""The CRT's stores at the edges of its waves (64 lanes of 4 rows): columns
shorter than a lane's rows, than a wave, one row past a wave, waves across
several columns and the last one's idle lanes, leading dimensions and first
entries at every alignment, and the moduli left over from groups of four.  Bit-
exact against the oracle; entries between the columns keep their value."""
import numpy as np
import pytest

from gpu_util import announce, host
from oracle.complex_gemm import os_ii_complex, os_ii_complex_3m
from oracle.ozaki2 import os_ii
from workload import complex_gemm_inputs, gemm_inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2602_02549_amd as oz  # noqa: E402

FORMS = {
    "dgemm": (oz.ozaki2_gemm, np.float64, os_ii),
    "sgemm": (oz.ozaki2_sgemm, np.float32, os_ii),
    "zgemm": (oz.ozaki2_zgemm, np.complex128, os_ii_complex),
    "cgemm": (oz.ozaki2_cgemm, np.complex64, os_ii_complex),
    "zgemm3m": (oz.ozaki2_zgemm3m, np.complex128, os_ii_complex_3m),
    "cgemm3m": (oz.ozaki2_cgemm3m, np.complex64, os_ii_complex_3m),
}


# N = 4 to 9: 0 to 3 moduli after whole groups of four
@pytest.mark.parametrize("m,n,N", [
    (1, 1, 4), (1, 300, 5), (3, 100, 6), (4, 64, 7), (5, 53, 8), (255, 3, 9), (256, 4, 5),
    (257, 3, 6), (1000, 2, 7), (1024, 1, 8),
])
@pytest.mark.parametrize("form", list(FORMS))
def test_crt_stores(form, m, n, N):
    call, dtype, oracle = FORMS[form]
    announce(f"crt {form} {m}x{n} N={N}")
    k = 12
    make = complex_gemm_inputs if np.dtype(dtype).kind == "c" else gemm_inputs
    A, B = make(m, n, k, phi=0.5, seed=m + n + N, dtype=dtype)
    want = oracle(A, B, N)
    dA = torch.from_numpy(np.ascontiguousarray(A.T)).to("cuda:0")
    dB = torch.from_numpy(np.ascontiguousarray(B.T)).to("cuda:0")
    for first, ldc in ((0, m), (1, m), (0, m + 1), (3, m + 2)):
        C = torch.full((first + n * ldc + 4,), 7.0, dtype=dA.dtype, device="cuda:0")
        rc = call(m, n, k, dA.data_ptr(), m, dB.data_ptr(), k,
                  C.data_ptr() + first * C.element_size(), ldc, N)
        assert rc == oz.OK
        got = host(C)
        ref = np.full(got.shape, 7.0, dtype)
        ref[first:first + n * ldc].reshape(n, ldc)[:, :m] = want.T
        assert np.array_equal(got, ref), (first, ldc)
    assert oz.ozaki2_sync_status() == oz.OK
