"""The scan with more workgroups than one grid dimension takes threads for: more
than 2^22 columns of B that take a workgroup each (2^22 workgroups are 2^31
threads), and more than 2^23 (2^32 threads, the most along one dimension).  The
columns repeat 64 different ones, so every column of C is the oracle's for those."""
import numpy as np
import pytest

from gpu_util import announce, dev
from oracle.ozaki2 import os_ii

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
import paper_2602_02549_amd as oz  # noqa: E402

M, K, N = 3, 2049, 2      # k > 2048: a workgroup a column


@pytest.mark.parametrize("n,batched", [((1 << 22) + 64, False), ((1 << 23) + 64, False),
                                       ((1 << 23) + 64, True)])
def test_many_columns(n, batched):
    announce(f"scan grid n={n} batched={batched}")
    rng = np.random.default_rng(n)
    A = (rng.random((M, K)) - 0.5).astype(np.float32)
    B64 = (rng.random((K, 64)) - 0.5).astype(np.float32)
    want = torch.from_numpy(np.ascontiguousarray(os_ii(A, B64, N).T)).cuda()      # (64, M)
    torch.cuda.empty_cache()
    need = (oz.ozaki2_batched_workspace_bytes(32, [M, n, K, N]) if batched
            else oz.ozaki2_workspace_bytes(32, M, n, K, N))
    ws = torch.empty(need + 256, dtype=torch.uint8, device="cuda")
    B = torch.from_numpy(np.ascontiguousarray(B64.T)).cuda().repeat(n // 64, 1)   # (n, K)
    C = torch.zeros(n, M, dtype=torch.float32, device="cuda")
    At = oz.col_major(dev(A))
    rc = oz.ozaki2_set_workspace(ws.data_ptr(), need)
    assert rc == oz.OK
    try:
        oz.ozaki2_set_stream(torch.cuda.current_stream().cuda_stream)
        if batched:
            oz.gemm_batched_cm([At], [B], [C], [(M, n, K)], [N])
        else:
            assert oz.ozaki2_sgemm(M, n, K, At.data_ptr(), M, B.data_ptr(), K, C.data_ptr(), M,
                                   N) == oz.OK
        torch.cuda.synchronize()
        assert bool((C.view(-1, 64, M) == want).all())
    finally:
        torch.cuda.synchronize()
        oz.ozaki2_set_workspace(0, 0)
        del ws, B, C
        torch.cuda.empty_cache()
