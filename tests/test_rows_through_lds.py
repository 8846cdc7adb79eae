"""Products whose waves bring k-contiguous operands in through LDS, two slabs (16 k in fp32, 32 in 16 bits) at a time: waves without a slab, with
an odd number of them and with more pairs than are in flight; rows further apart than they are long; segments that no pair is a
multiple of."""
import numpy as np
import pytest
import torch

import paper_2507_10392_amd as zs
from harness import dev, log_report, rel_err
from workloads import round_bf16, round_f16

pytestmark = pytest.mark.gpu
TD = {0: torch.float32, 1: torch.bfloat16, 2: torch.float16}
ROUND = {0: lambda a: a, 1: round_bf16, 2: round_f16}
TOL = {0: 2e-5, 1: 2.0 ** -8, 2: 2.0 ** -11}     # the bar of the other fp32 products; one rounding of the largest value
# fp32: outputs that take 16x16, 16x32, 32x32 (K over 8 waves) and 64x64 tiles (K over 4) at each of these K, the larger ones as one round of
# 256 workgroups; 16 bits: input gradients on 32x32 and 64x64 (K over 8)
OUTPUTS = [(0, 36, 40), (0, 100, 776), (0, 250, 1000), (0, 500, 2020), (1, 36, 40), (1, 260, 520), (1, 1000, 1016), (2, 36, 40), (2, 1000, 1016)]
DEPTHS = [8, 40, 264, 528, 1304, 2720]


@pytest.mark.parametrize("K", DEPTHS)
@pytest.mark.parametrize("dtype,M,N", OUTPUTS)
def test_forward_input_gradient_and_segments(gpu_device, dtype, M, N, K):
    print(f"[case] rows through LDS dtype={dtype} M={M} N={N} K={K}", flush=True)
    rng = np.random.default_rng(71)
    st = torch.cuda.current_stream().cuda_stream
    td = TD[dtype]
    lda, ldb, kseg = K + 16, K + 24, K // 2 if K % 16 == 0 else K
    A, B = (ROUND[dtype](rng.standard_normal((r, w)).astype(np.float32)) for r, w in ((M, lda), (N, ldb)))
    A[:, K:] = B[:, K:] = np.nan               # between the rows
    want = A[:, :K].astype(np.float64) @ B[:, :K].astype(np.float64).T
    S = np.ascontiguousarray(B[:, :K].reshape(N, K // kseg, kseg).transpose(1, 0, 2))
    errs = []
    for name, tb, b, ld, seg in (("nn", 0, np.ascontiguousarray(B[:, :K].T), N, 0), ("nt", 1, B, ldb, 0), ("segments", 1, S, kseg, kseg)):
        C = torch.full((M, N), float("nan"), dtype=td, device="cuda")
        zs.ops.gemm(st, dtype, 0, tb, M, N, K, dev(A, td), lda, dev(b, td), ld, C, N, 0, None, None, 0, 1, 0, 0, 0, 0, seg, N * kseg if seg else 0, 0)
        torch.cuda.synchronize()
        errs.append((name, rel_err(C.float().cpu().numpy().astype(np.float64), want)))
    log_report(f"rows through LDS {dtype} {M} {N} {K}", errs)
    assert all(e <= TOL[dtype] for _, e in errs), errs
