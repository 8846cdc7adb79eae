"""fp32 products on 16x16, 16x32 and 32x32 tiles on both sides of the rule that brings k-contiguous operands in directly or through LDS: the same
bits whether rows are whole lines or not, and float64's values."""
import numpy as np
import pytest
import torch

import paper_2507_10392_amd as zs
from harness import dev, rel_err

pytestmark = pytest.mark.gpu
SIZES = [(40, 72, k) for k in (8, 64, 72, 128, 136)] + [(200, 512, k) for k in (64, 68, 128)] + [(300, 640, k) for k in (60, 68, 328, 388, 1384, 1660)] + \
        [(128, 1024, 1020), (128, 1024, 1036)]


@pytest.mark.parametrize("M,N,K", SIZES)
@pytest.mark.parametrize("tb", [0, 1])
def test_same_bits_with_rows_that_are_whole_lines(gpu_device, M, N, K, tb):
    print(f"[case] fp32 product both ways M={M} N={N} K={K} transposed={tb}", flush=True)
    rng = np.random.default_rng(97)
    st = torch.cuda.current_stream().cuda_stream
    A, B = rng.standard_normal((M, K)).astype(np.float32), rng.standard_normal((K, N)).astype(np.float32)
    want = A.astype(np.float64) @ B.astype(np.float64)
    got = []
    for ld in (-(-K // 32) * 32, -(-K // 32) * 32 + 4):
        a = torch.full((M, ld), float("nan"), device="cuda")
        a[:, :K] = dev(A)
        b = dev(B)
        if tb:
            b = torch.full((N, ld), float("nan"), device="cuda")
            b[:, :K] = dev(np.ascontiguousarray(B.T))
        C = torch.full((M, N), float("nan"), device="cuda")
        zs.ops.gemm(st, 0, 0, tb, M, N, K, a, ld, b, ld if tb else N, C, N, 0, None, None, 0, 1, 0, 0, 0, 0, 0, 0, 0)
        torch.cuda.synchronize()
        got.append(C.cpu().numpy())
    assert rel_err(got[0], want) <= 2e-5                      # the bar of the other fp32 products
    assert np.array_equal(got[0], got[1])
