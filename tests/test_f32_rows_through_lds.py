"""fp32 products whose waves bring k-contiguous operands in through LDS, two slabs of 16 k at a time: waves without a slab, with an odd number of
them and with more pairs than are in flight; rows further apart than they are long; segments that no pair is a multiple of."""
import numpy as np
import pytest
import torch

import paper_2507_10392_amd as zs
from harness import dev, log_report, rel_err

pytestmark = pytest.mark.gpu
# outputs that take 16x16, 16x32, 32x32 (K over 8 waves) and 64x64 tiles (K over 4)
OUTPUTS = [(36, 40), (100, 776), (260, 1032), (520, 2052)]


@pytest.mark.parametrize("K", [4, 36, 260, 540, 1300])
@pytest.mark.parametrize("M,N", OUTPUTS)
def test_forward_input_gradient_and_segments(gpu_device, M, N, K):
    print(f"[case] fp32 rows through LDS M={M} N={N} K={K}", flush=True)
    rng = np.random.default_rng(71)
    st = torch.cuda.current_stream().cuda_stream
    lda, ldb, kseg = K + 12, K + 20, K // 2 if K % 8 == 0 else K // 4 if K % 16 == 0 else K
    A, B = rng.standard_normal((M, lda)).astype(np.float32), rng.standard_normal((N, ldb)).astype(np.float32)
    A[:, K:] = B[:, K:] = np.nan               # between the rows
    want = A[:, :K].astype(np.float64) @ B[:, :K].astype(np.float64).T
    S = np.ascontiguousarray(B[:, :K].reshape(N, K // kseg, kseg).transpose(1, 0, 2))
    errs = []
    for name, tb, b, ld, seg in (("nn", 0, np.ascontiguousarray(B[:, :K].T), N, 0), ("nt", 1, B, ldb, 0), ("segments", 1, S, kseg, kseg)):
        C = torch.full((M, N), float("nan"), device="cuda")
        zs.ops.gemm(st, 0, 0, tb, M, N, K, dev(A), lda, dev(b), ld, C, N, 0, None, None, 0, 1, 0, 0, 0, 0, seg, N * kseg if seg else 0, 0)
        torch.cuda.synchronize()
        errs.append((name, rel_err(C.cpu().numpy().astype(np.float64), want)))
    log_report(f"fp32 rows through LDS {M} {N} {K}", errs)
    assert all(e <= 2e-5 for _, e in errs), errs     # the bar of the other fp32 products
