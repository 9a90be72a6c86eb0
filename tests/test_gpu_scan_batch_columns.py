"""The scan of a batch of many workgroups where a column goes from a wave to a workgroup
(32 KB: 4096 of k in FP64, 8192 in FP32), with columns beyond what a wave keeps in
registers: every problem as the oracle."""
import numpy as np
import pytest

from gpu_util import announce, dev, host
from oracle.ozaki2 import os_ii
from workload import gemm_inputs

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2602_02549_amd as oz  # noqa: E402


@pytest.mark.parametrize("dtype,ks", [(np.float64, (2048, 2049, 4096, 4097)),
                                      (np.float32, (2049, 8192, 8193, 5000))])
def test_columns(dtype, ks):
    announce(f"batch columns {np.dtype(dtype).name}")
    count, N = 48, 5
    shapes = [(3 + p % 4, 1 + 37 * (p % 5), ks[p % 4]) for p in range(count)]
    ins = [gemm_inputs(m, n, k, phi=1.0, seed=p, dtype=dtype) for p, (m, n, k) in enumerate(shapes)]
    for a, b in ins:
        b[-1, 0] *= 64             # the maximum of a column in its last element
    got = oz.gemm_batched([dev(a) for a, _ in ins], [dev(b) for _, b in ins], [N] * count)
    for (a, b), c in zip(ins, got):
        assert np.array_equal(host(c), os_ii(a, b, N))
