"""Residue slices at the edges of their kernel, every stage bit-exact against
the oracle: both ends of each residue path (limbs, exact steps) on entries
whose scaled integers sit on limb boundaries and on ties, and launches with
few tiles, whose moduli are dealt to several workgroups per tile (from one
tile to just past the point where every tile has one workgroup)."""
import numpy as np
import pytest

from gpu_util import announce, compare_stages, dev, host
from oracle.ozaki2 import os_ii

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2602_02549_amd as oz  # noqa: E402


def edge_matrix(rng, shape):
    """Powers of two, their neighbours, and odd multiples of 2^-j (ties of every
    split at 2^40, 2^48 or 2^80), with signs, one entry of size 1 per row."""
    j = rng.integers(0, 60, shape)
    base = np.ldexp(1.0, -j)
    kind = rng.integers(0, 4, shape)
    X = np.where(kind == 0, base, np.where(kind == 1, base * (1 - 2.0 ** -53),
                 np.where(kind == 2, base * (1 + 2.0 ** -52), base * 1.5)))
    X = X * rng.choice([-1.0, 1.0], shape)
    X[rng.random(shape) < 0.1] = 0.0
    return X


def check(A, B, N, what):
    announce(f"residue edges {what} {A.shape} x {B.shape} N={N}")
    got = {kk: host(v) for kk, v in oz.debug_stages(dev(A), dev(B), N).items()}
    C_ref, st = os_ii(A, B, N, stages=True)
    assert compare_stages(got, st, C_ref, N) == []
    assert oz.ozaki2_sync_status() == oz.OK


@pytest.mark.parametrize("N", [2, 3, 11, 12, 22, 23, 31, 32, 40, 41, 49])
def test_residue_paths_on_limb_boundaries(N):
    rng = np.random.default_rng(N)
    check(edge_matrix(rng, (33, 130)), edge_matrix(rng, (130, 20)), N, "FP64")


@pytest.mark.parametrize("N", [2, 7, 11, 12, 16])
def test_residue_paths_on_limb_boundaries_fp32(N):
    rng = np.random.default_rng(100 + N)
    A = edge_matrix(rng, (33, 130)).astype(np.float32)
    B = edge_matrix(rng, (130, 20)).astype(np.float32)
    check(A, B, N, "FP32")


# tiles are 32 rows x 128 k; N moduli are dealt to min(N / 2, 512 / tiles) workgroups per tile
@pytest.mark.parametrize("m,n,k,N", [
    (1, 1, 1, 2), (32, 32, 128, 3), (33, 64, 129, 15), (100, 300, 700, 14),
    (512, 31, 1024, 14), (520, 40, 1900, 5), (544, 33, 2048, 13),
])
def test_tiles_shared_by_workgroups(m, n, k, N):
    rng = np.random.default_rng(m + n + k)
    check(rng.standard_normal((m, k)), rng.standard_normal((k, n)), N, "shared tiles")
