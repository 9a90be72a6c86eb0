"""The scan of few strips where its route changes with the number of passes: FP32
(strips of 32 rows, 256 of k a pass) at 8 and 9 passes with few columns (strips, then
chunks), at 9 passes with 2735 and 2736 columns (chunks, then strips) and at 16 and
17; single calls stage by stage, complex calls and batches against the oracle."""
import numpy as np
import pytest

from gpu_util import announce, compare_stages, dev, host
from oracle.complex_gemm import os_ii_complex, os_ii_complex_3m
from oracle.ozaki2 import os_ii
from workload import complex_gemm_inputs, gemm_inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2602_02549_amd as oz  # noqa: E402


@pytest.mark.parametrize("m,n,k", [(33, 5, 2048), (33, 5, 2049), (5, 2735, 2304), (5, 2736, 2304),
                                   (33, 5, 4096)])
def test_passes(m, n, k):
    announce(f"scan passes {m}x{n}x{k}")
    N = 3
    A, B = gemm_inputs(m, n, k, phi=1.0, seed=m + n + k, dtype=np.float32)
    A[0, k - 1] *= 64
    B[k - 1, 0] *= 64
    got = {kk: host(v) for kk, v in oz.debug_stages(dev(A), dev(B), N, crt_stages=False).items()}
    C_ref, st = os_ii(A, B, N, stages=True)
    assert compare_stages(got, st, C_ref, N) == []


@pytest.mark.parametrize("form,oracle", [("4m", os_ii_complex), ("3m", os_ii_complex_3m)])
@pytest.mark.parametrize("m,n,k", [(33, 5, 2048), (33, 5, 2049), (9, 2736, 2304), (40, 7, 4096)])
def test_passes_complex(form, oracle, m, n, k):
    announce(f"scan passes {form} {m}x{n}x{k}")
    N = 5
    A, B = complex_gemm_inputs(m, n, k, phi=1.0, seed=m + n + k)
    A, B = A.astype(np.complex64), B.astype(np.complex64)
    rows, cols = np.array([0, m // 2, m - 1]), np.array([0, n // 2, n - 1])
    got = host(oz.zgemm(dev(A), dev(B), N, form=form))
    assert np.array_equal(got[np.ix_(rows, cols)], oracle(A, B, N, rows=rows, cols=cols))


@pytest.mark.parametrize("count", [2, 40])     # few workgroups, and many
def test_passes_batched(count):
    announce(f"scan passes batch of {count}")
    N = 5
    shapes = [(33 + 8 * (p % 3), 5 + 16 * (p % 5), (2049, 2048, 2305, 4096, 4097)[p % 5])
              for p in range(count)]
    ins = [gemm_inputs(m, n, k, phi=1.0, seed=p, dtype=np.float32)
           for p, (m, n, k) in enumerate(shapes)]
    got = oz.gemm_batched([dev(a) for a, _ in ins], [dev(b) for _, b in ins], [N] * count)
    for (a, b), c in zip(ins, got):
        assert np.array_equal(host(c), os_ii(a, b, N))
