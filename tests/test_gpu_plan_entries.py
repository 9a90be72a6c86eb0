"""The planner's and the certificate's passes over the entries (waves of 64 lanes
with four rows each) where the rows do not fill a lane, a wave or a second one,
the entry that decides lies in the last rows, and exact zeros lie beside it:
against the oracle's bracket for N and its ratio, as the larger cases are."""
import numpy as np
import pytest

from gpu_util import announce, dev, host
from oracle.bounds import certified_ratio, planner_terms, required_moduli_from_terms
from oracle.ozaki2 import os_ii
from workload import gemm_inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2602_02549_amd as oz  # noqa: E402


def slack(k):
    # the lower bound of S: BF16 operands rounded down (2^-7 each), FP32 sums of k terms
    return 2.0 ** -6 + k * 2.0 ** -22 + 1e-9


def inputs(m, n, k):
    A, B = gemm_inputs(m, n, k, phi=0.5, seed=m + n + k)
    A[m - 1] *= np.exp2(np.linspace(0, 30, k))    # the last row needs more moduli
    if m > 2:
        A[m - 2] = 0.0
    if n > 2:
        B[:, n - 2] = 0.0
    return A, B


SHAPES = [(1, 1, 20), (3, 2, 40), (4, 9, 40), (5, 1, 40), (255, 4, 30), (256, 3, 30), (257, 5, 30),
          (261, 70, 30), (513, 2, 30)]


@pytest.mark.parametrize("m,n,k", SHAPES)
def test_required_moduli_edges(m, n, k):
    announce(f"plan entries {m}x{n}x{k}")
    A, B = inputs(m, n, k)
    rc, Ng = oz.required_moduli(dev(A), dev(B), 1e-13)
    terms = planner_terms(A, B)
    lo = required_moduli_from_terms(terms, 1e-13 * (1 + 1e-9))
    hi = required_moduli_from_terms(terms, 1e-13 * (1 - slack(k)))
    g = Ng if rc == oz.OK else 50
    assert rc in (oz.OK, oz.ERR_UNREACHABLE)
    assert (lo[0] if lo[1] else 50) <= g <= (hi[0] if hi[1] else 50)


@pytest.mark.parametrize("m,n,k", SHAPES)
def test_certified_ratio_edges(m, n, k):
    announce(f"certify {m}x{n}x{k}")
    A, B = inputs(m, n, k)
    N = 14
    C, rc, N_used, ratio = oz.gemm_certified(dev(A), dev(B), 1.0, N)
    assert rc == oz.OK and N_used == N
    C_ref, st = os_ii(A, B, N, stages=True)
    assert np.array_equal(host(C), C_ref)
    want = certified_ratio(A, B, st)
    assert want * (1 - 1e-12) <= ratio <= want / (1 - slack(k))
