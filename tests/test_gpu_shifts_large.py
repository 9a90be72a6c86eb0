"""The shifts at maxima of Cbar from 10^6 to past 2 10^9, where FP32 rounds the maximum
up (from 2^24 on): rows whose maximum is the first at a step, or the one before, against
the oracle."""
import numpy as np
import pytest

from gpu_util import announce, dev, host
from oracle.constants import constants
from oracle.ozaki2 import shift
from test_gpu_shifts import steps

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2602_02549_amd as oz  # noqa: E402

K = 519_000          # 4096 (K - 1) is the largest maximum


def row_with_maximum(M):
    """A row (abs max 127/64, so mu' = 5 and bar 64) whose Cbar against the column (127/64,
    ..., 127/64, 1/32), bars 64 ... 64 1, is M >= 4096."""
    a = np.zeros(K)
    full, rest = divmod(M, 64 * 64)
    a[:full] = 127.0 / 64
    a[full] = rest // 64 / 32.0
    a[K - 1] = rest % 64 / 32.0
    return a


@pytest.mark.parametrize("prec,N,table", [(64, 2, "paper"), (64, 14, "paper"), (64, 49, "optimal"),
                                          (32, 7, "paper")])
def test_large_maxima(prec, N, table):
    const = constants(N, prec, table)
    at = steps(const, 10 ** 6, 4096 * (K - 2))
    assert len(at) >= 5 and at[-1] > 2 ** 24, at
    targets = sorted({m for s in at for m in (s - 1, s)} | {2 ** 24 + 1, 4096 * (K - 2)})
    announce(f"large shifts b={prec} N={N} {table} M={targets}")
    dt = np.float64 if prec == 64 else np.float32
    A = np.stack([row_with_maximum(M) for M in targets]).astype(dt)
    B = np.full((K, 1), 127.0 / 64, dtype=dt)
    B[K - 1] = 1.0 / 32
    with oz.moduli_table(oz.MODULI_PAPER if table == "paper" else oz.MODULI_OPTIMAL):
        got = oz.debug_stages(dev(A), dev(B), N, crt_stages=False)
    assert host(got["rmax"]).tolist() == targets
    assert host(got["mu"]).tolist() == [shift(5, M, const) for M in targets]
    assert host(got["nu"]).tolist() == [shift(5, max(targets), const)]
