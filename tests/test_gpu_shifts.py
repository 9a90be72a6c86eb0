"""The shifts mu, nu of Algorithm 2 at the maxima of Cbar where they step:
rows whose maximum is the first at a step, or the one before, against the
oracle's log2f and floor."""
import numpy as np
import pytest

from gpu_util import announce, dev, host
from oracle.constants import constants
from oracle.ozaki2 import shift

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2602_02549_amd as oz  # noqa: E402

K = 16500            # 32 * 32 + 64 * (K - 1) covers maxima up to 1.05e6


def steps(const, lo, hi):
    """The M in (lo, hi] at which shift(0, M) first takes a smaller value."""
    out = []
    at, M = shift(0, lo, const), lo
    while shift(0, hi, const) < at:
        a, b = M, hi                      # shift(a) = at > shift(b)
        while b - a > 1:
            mid = (a + b) // 2
            if shift(0, mid, const) == at:
                a = mid
            else:
                b = mid
        out.append(b)
        at, M = shift(0, b, const), b
    return out


def row_with_maximum(M):
    """A row of A (abs max in [1, 2), so mu' = 5) whose Cbar against the column
    (1, 1/32, 1/32, ...) is M: bars 32 32 + sum of bars 1..64 times 1."""
    a = np.zeros(K)
    a[0] = 1.0
    rest = M - 32 * 32
    full, part = divmod(rest, 64)
    a[1:1 + full] = 127.0 / 64            # bar ceil(63.5) = 64
    if part:
        a[1 + full] = part / 32.0 if part < 64 else 0.0
    return a


@pytest.mark.parametrize("prec,N,table", [(64, 2, "paper"), (64, 3, "paper"), (64, 14, "paper"),
                                          (64, 30, "optimal"), (64, 49, "paper"), (32, 7, "paper"),
                                          (32, 16, "optimal")])
def test_shift_steps(prec, N, table):
    const = constants(N, prec, table)
    at = steps(const, 1025, 32 * 32 + 64 * (K - 2))
    assert len(at) >= 4, at
    targets = sorted({m for s in at for m in (s - 1, s)} | {1024, 1025})
    announce(f"shift steps b={prec} N={N} {table} M={targets}")
    dt = np.float64 if prec == 64 else np.float32
    A = np.stack([row_with_maximum(M) for M in targets]).astype(dt)
    B = np.full((K, 1), 1.0 / 32)
    B[0] = 1.0
    with oz.moduli_table(oz.MODULI_PAPER if table == "paper" else oz.MODULI_OPTIMAL):
        got = oz.debug_stages(dev(A), dev(B.astype(dt)), N, crt_stages=False)
    assert host(got["rmax"]).tolist() == targets
    assert host(got["mu"]).tolist() == [shift(5, M, const) for M in targets]
    assert host(got["nu"]).tolist() == [shift(5, max(targets), const)]
