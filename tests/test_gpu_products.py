"""The matrix-core products at the edges of their launches: a last round of few
256 x 256 tiles cut into two or four parts, the ring of four group buffers that
launches of at most one 128 x 128 tile per compute unit use (from one group of
k to more than the ring holds), and split products whose last rows and columns
are padding.  All bit-exact: against the 128 x 128 tiles, the unsplit products
and the oracle."""
import numpy as np
import pytest

from gpu_util import announce, compare_stages, dev, host
from oracle.ozaki2 import os_ii
from workload import gemm_inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2602_02549_amd as oz  # noqa: E402


def with_knob(knob, value, f):
    rc, prev = oz.ozaki2_debug_tuning(knob, value)
    assert rc == oz.OK
    try:
        return f()
    finally:
        oz.ozaki2_debug_tuning(knob, prev)


# 16 tiles of 256 x 256 per modulus: 272 and 320 tiles (last round of 16 and 64:
# four parts), 352 and 384 (96 and 128: two parts), 256 and 400 (0 and 144: none)
@pytest.mark.parametrize("m,n,k,N", [
    (1024, 1024, 200, 17), (1000, 1010, 130, 20), (1024, 1020, 129, 22), (1001, 1024, 300, 24),
    (1024, 1024, 128, 16), (1024, 1024, 128, 25),
])
def test_last_round_in_parts(m, n, k, N):
    announce(f"parts {m}x{n}x{k} N={N}")
    A, B = gemm_inputs(m, n, k, phi=0.5, seed=m + n + k + N)
    dA, dB = dev(A), dev(B)
    got = host(oz.gemm(dA, dB, N))
    assert np.array_equal(got, host(with_knob(oz.KNOB_GEMM_TILE, 2, lambda: oz.gemm(dA, dB, N))))
    # entries of every quarter of the last tile, whose modulus is the last one
    rows = np.array([0, m // 2, m - 200, m - 1])
    cols = np.array([0, n // 2, n - 200, n - 1])
    assert np.array_equal(got[np.ix_(rows, cols)], os_ii(A, B, N, rows=rows, cols=cols))
    assert oz.ozaki2_sync_status() == oz.OK


# one to nine groups of 128 k in a ring of four; from eight on two splits
@pytest.mark.parametrize("k", [1, 128, 129, 300, 512, 513, 640, 1100])
@pytest.mark.parametrize("m,n", [(60, 50), (129, 257)])
def test_ring_stages(m, n, k):
    announce(f"ring {m}x{n}x{k}")
    N = 3
    A, B = gemm_inputs(m, n, k, phi=1.0, seed=m + n + k)
    got = {kk: host(v) for kk, v in oz.debug_stages(dev(A), dev(B), N).items()}
    C_ref, st = os_ii(A, B, N, stages=True)
    assert compare_stages(got, st, C_ref, N) == []


# one row past a tile, one short of it, and a few rows of one
@pytest.mark.parametrize("m,n,k,N", [(129, 127, 4500, 4), (5, 130, 9000, 3), (256, 3, 4096, 3)])
def test_split_padding(m, n, k, N):
    announce(f"split padding {m}x{n}x{k} N={N}")
    A, B = gemm_inputs(m, n, k, phi=1.0, seed=m + n + k)
    dA, dB = dev(A), dev(B)
    got = {kk: host(v) for kk, v in oz.debug_stages(dA, dB, N).items()}
    C_ref, st = os_ii(A, B, N, stages=True)
    assert compare_stages(got, st, C_ref, N) == []
    one = host(with_knob(oz.KNOB_SPLIT_K, 1, lambda: oz.gemm(dA, dB, N)))
    assert np.array_equal(host(oz.gemm(dA, dB, N)), one)
