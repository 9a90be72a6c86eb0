"""The scan (abs-max and bars) at the edges of its split, every stage bit-exact
against the oracle: strips of 64, 32 and 16 rows (k to 128, 256 and beyond),
ragged strips, chunks of k kept in registers and read again, columns on 4 to
64 lanes and on a workgroup, the chunked scan of long operands, and the same
through a batch (whose split depends on the whole batch)."""
import numpy as np
import pytest

from gpu_util import announce, compare_stages, dev, host
from oracle.ozaki2 import os_ii

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2602_02549_amd as oz  # noqa: E402


def matrices(m, n, k, dtype):
    """Normal entries times a random power of two per row and column, with zeros,
    one zero row and one zero column."""
    rng = np.random.default_rng(m * 7 + n * 3 + k)
    A = np.ldexp(rng.standard_normal((m, k)), rng.integers(-20, 20, (m, 1)))
    B = np.ldexp(rng.standard_normal((k, n)), rng.integers(-20, 20, (1, n)))
    A[rng.random(A.shape) < 0.05] = 0.0
    A[m // 2] = 0.0
    B[:, n // 2] = 0.0
    return A.astype(dtype), B.astype(dtype)


SHAPES = [
    # k_pad 128, 256, 384, 512, 640: the strip heights, and one or two chunks
    (65, 33, 1), (70, 40, 128), (33, 30, 129), (17, 20, 256), (48, 17, 300), (31, 33, 512),
    (30, 20, 513),
    # a chunk past the two in registers; the last chunk one k long
    (20, 9, 1025), (33, 12, 1600),
    # columns: the last length of a wave, the first of a workgroup, past its registers
    (10, 9, 2048), (9, 10, 2049), (7, 5, 16385),
    # few strips over a long k: chunked; enough rows for strips again (96 strips of 16)
    (40, 6, 4097), (1537, 3, 4100),
]


@pytest.mark.parametrize("dtype", [np.float64, np.float32])
@pytest.mark.parametrize("m,n,k", SHAPES)
def test_scan_stages(m, n, k, dtype):
    announce(f"scan {m}x{n}x{k} {np.dtype(dtype).name}")
    A, B = matrices(m, n, k, dtype)
    N = 3
    got = {kk: host(v) for kk, v in oz.debug_stages(dev(A), dev(B), N, crt_stages=False).items()}
    C_ref, st = os_ii(A, B, N, stages=True)
    assert compare_stages(got, st, C_ref, N) == []
    assert oz.ozaki2_sync_status() == oz.OK


@pytest.mark.parametrize("count", [1, 60])      # a fine and a coarse split
def test_scan_in_a_batch(count):
    shapes = (SHAPES * count)[:max(len(SHAPES), count * 3)]
    announce(f"scan in a batch of {len(shapes)}")
    pairs = [matrices(m, n, k, np.float64) for m, n, k in shapes]
    Ns = [3 + i % 3 for i in range(len(shapes))]
    got = oz.gemm_batched([dev(A) for A, _ in pairs], [dev(B) for _, B in pairs], Ns)
    ref = {}
    for i, ((A, B), N) in enumerate(zip(pairs, Ns)):
        key = (shapes[i], N)
        if key not in ref:
            ref[key] = os_ii(A, B, N)
        assert np.array_equal(host(got[i]), ref[key]), (i, key)


@pytest.mark.parametrize("form", ["4m", "3m"])
@pytest.mark.parametrize("m,n,k", [(65, 33, 100), (33, 20, 300), (20, 9, 700), (9, 10, 1100),
                                   (6, 5, 2100), (40, 3, 4100)])
def test_scan_of_complex_operands(form, m, n, k):
    from oracle.complex_gemm import os_ii_complex, os_ii_complex_3m
    announce(f"scan complex {form} {m}x{n}x{k}")
    Ar, Br = matrices(m, n, k, np.float64)
    Ai, Bi = matrices(m + 0, n, k, np.float64)
    A, B = Ar + 1j * np.roll(Ai, 1, axis=0), Br + 1j * np.roll(Bi, 1, axis=1)
    got = host(oz.zgemm(dev(A), dev(B), 4, form=form))
    ref = (os_ii_complex if form == "4m" else os_ii_complex_3m)(A, B, 4)
    assert np.array_equal(got, ref[0] if isinstance(ref, tuple) else ref)


def test_nonfinite_rows_and_columns_are_found():
    for where in ("A", "B"):
        for bad in (np.inf, -np.inf, np.nan):
            for k in (100, 5000):
                A, B = matrices(40, 6, k, np.float64)
                (A if where == "A" else B)[(-1, k - 1) if where == "A" else (k - 1, -1)] = bad
                announce(f"scan non-finite {where} {bad} k={k}")
                C = host(oz.gemm(dev(A), dev(B), 5))
                assert np.isnan(C).all()
                assert oz.ozaki2_sync_status() == oz.ERR_NONFINITE
    A, B = matrices(40, 6, 100, np.float64)
    assert np.isfinite(host(oz.gemm(dev(A), dev(B), 5))).all()
    assert oz.ozaki2_sync_status() == oz.OK
