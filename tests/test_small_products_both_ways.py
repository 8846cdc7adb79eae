"""16-bit products on small tiles on both sides of the rules that share a tile's loads among waves or bring rows in through LDS: the bits do
not depend on the way."""
import numpy as np
import pytest
import torch

import paper_2507_10392_amd as zs

pytestmark = pytest.mark.gpu
TD = {1: torch.bfloat16, 2: torch.float16}
nan = float("nan")
GRADIENTS, DEPTHS = [(70, 136), (1000, 1016)], [8, 248, 256, 264, 512, 760, 768, 776, 1280]
# 252, 256, 288, 308, 319 and 464 tiles of 32x32; rows of x that are whole lines (K = 512, 768) and that are not
FORWARDS = [(200, 1152, 96), (500, 512, 512), (230, 1152, 64), (230, 1152, 96), (230, 1152, 104), (330, 904, 256), (330, 904, 264), (330, 904, 768),
            (330, 896, 776), (500, 904, 256), (500, 904, 264), (500, 904, 512), (330, 904, 2600), (330, 904, 2616)]


def padded(a, ld):
    """The same rows, ld elements apart."""
    out = torch.full((a.shape[0], ld), nan, dtype=a.dtype, device="cuda")
    out[:, :a.shape[1]] = a
    return out


def random(seed, td):
    g = torch.Generator(device="cuda").manual_seed(seed)
    return lambda *s: (torch.randn(s, generator=g, device="cuda") * 0.25).to(td)


# input gradients, whole and in two segments, with rows that are whole lines and rows that are not: 32x32 and 64x64 tiles
@pytest.mark.parametrize("dtype", [1, 2])
@pytest.mark.parametrize("M,N", GRADIENTS)
@pytest.mark.parametrize("K", DEPTHS)
def test_input_gradients_have_the_same_bits(gpu_device, dtype, M, N, K):
    print(f"[case] small input gradient both ways M={M} N={N} K={K} dtype={dtype}", flush=True)
    st, td = torch.cuda.current_stream().cuda_stream, TD[dtype]
    rnd = random(101, td)
    A, B = rnd(M, K), rnd(N, K)
    whole, out = -(-K // 64) * 64, []
    want = A.double() @ B.double().t()
    for lda, ldb in ((whole, whole), (whole + 8, whole + 16)):
        C = torch.full((M, N), nan, dtype=td, device="cuda")
        zs.ops.gemm(st, dtype, 0, 1, M, N, K, padded(A, lda), lda, padded(B, ldb), ldb, C, N, 0, None, None, 0, 1, 0, 0, 0, 0, 0, 0, 0)
        if K % 16 == 0:
            h = K // 2
            S = torch.stack([padded(B[:, :h], ldb), padded(B[:, h:], ldb)])
            C2 = torch.full_like(C, nan)
            zs.ops.gemm(st, dtype, 0, 1, M, N, K, padded(A, lda), lda, S, ldb, C2, N, 0, None, None, 0, 1, 0, 0, 0, 0, h, N * ldb, 0)
            torch.cuda.synchronize()
            assert torch.equal(C2.view(torch.int16), C.view(torch.int16))
        torch.cuda.synchronize()
        out.append(C)
    assert torch.equal(out[0].view(torch.int16), out[1].view(torch.int16))
    # sums of K products of 16-bit values in fp32, one rounding of the result
    assert float((out[0].double() - want).abs().max() / want.abs().max()) <= {1: 2.0 ** -8, 2: 2.0 ** -11}[dtype]


# against the staged kernels' bits: plain, rotated, and the gated unit
@pytest.mark.parametrize("dtype", [1, 2])
@pytest.mark.parametrize("M,N,K", FORWARDS)
def test_forward_products_have_the_staged_kernels_bits(gpu_device, dtype, M, N, K):
    print(f"[case] small forward both ways M={M} N={N} K={K} dtype={dtype}", flush=True)
    st, td = torch.cuda.current_stream().cuda_stream, TD[dtype]
    rnd = random(103, td)
    A, W, bias, R = rnd(M, K), rnd(2, K, N), rnd(N), rnd(M, N)
    table = torch.empty(M, 64, 2, device="cuda")
    zs.ops.rope_table(st, M, 128, 10000.0, table)
    results = []
    for impl in (0, 2):
        C, rot, gu, a = (torch.full(s, nan, dtype=td, device="cuda") for s in ((M, N), (M, N // 128 * 128), (M, 2 * N), (M, N)))
        zs.ops.gemm(st, dtype, 0, 0, M, N, K, A, K, W, N, C, N, 0, bias, R, N, 1, 0, 0, 0, 0, 0, 0, impl)
        n = N // 128 * 128
        zs.ops.gemm_rope(st, dtype, 0, 0, M, n, K, A, K, W, N, rot, n, 0, None, None, 0, 1, 0, 0, 0, 0, 0, 0, impl, table, M, 128, 1)
        zs.ops.gemm_glu(st, dtype, 1, M, N, K, A, K, W, N, K * N, a, gu, impl)
        torch.cuda.synchronize()
        results.append((C, rot, gu, a))
    for name, x, y in zip(("plain", "rotated", "gate and up", "gated"), *results):
        assert not torch.isnan(x).any() and torch.equal(x.view(torch.int16), y.view(torch.int16)), name


# Forward products whose lines of W lie so far apart that the lines past K, which fill up a stage, would wrap around in 32 bits are for the
# staged tiles.  W's buffer is 256 MiB.
FAR_M, FAR_N, FAR_K = 40, 72, 16
FAR = [(2 ** 23 - 8, 32), (2 ** 23, 128)]


@pytest.mark.parametrize("dtype", [1, 2])
def test_forward_products_with_lines_far_apart(gpu_device, dtype):
    print(f"[case] lines far apart dtype={dtype}", flush=True)
    st, td = torch.cuda.current_stream().cuda_stream, TD[dtype]
    rnd = random(107, td)
    A, W, out = rnd(FAR_M, FAR_K), rnd(FAR_K, FAR_N), []
    for ldb, _ in FAR:
        far = torch.full((FAR_K * ldb,), nan, dtype=td, device="cuda")
        far.as_strided((FAR_K, FAR_N), (ldb, 1)).copy_(W)
        C = torch.full((FAR_M, FAR_N), nan, dtype=td, device="cuda")
        zs.ops.gemm(st, dtype, 0, 0, FAR_M, FAR_N, FAR_K, A, FAR_K, far, ldb, C, FAR_N, 0, None, None, 0, 1, 0, 0, 0, 0, 0, 0, 0)
        torch.cuda.synchronize()
        out.append(C)
    want = A.double() @ W.double()
    assert float((out[0].double() - want).abs().max() / want.abs().max()) <= {1: 2.0 ** -8, 2: 2.0 ** -11}[dtype]
    assert torch.equal(out[0].view(torch.int16), out[1].view(torch.int16))
