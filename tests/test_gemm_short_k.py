"""16-bit products on 128x128 tiles whose K has few 64-wide slabs: the K loop loads nothing past the last pair of slabs, so one, two,
three and more pairs take different ways through it.  Every output has to be the bits of the 256x256 tile, held against float64
elsewhere, which adds the same products in the same order."""
import pytest
import torch

import paper_2507_10392_amd as zs

pytestmark = pytest.mark.gpu
TD = {1: torch.bfloat16, 2: torch.float16}
SQUARE, SMALL = 3, 4      # impl: 256x256, 128x128


def st():
    return torch.cuda.current_stream().cuda_stream


def both(call, out):
    first = out.clone()
    call(SMALL, first)
    call(SQUARE, out)
    torch.cuda.synchronize()
    assert torch.isfinite(first.float()).all()
    assert torch.equal(first.view(torch.uint8), out.view(torch.uint8))


@pytest.mark.parametrize("dtype", [1, 2])
@pytest.mark.parametrize("K", [8, 64, 72, 128, 136, 192, 256, 264, 384, 448, 520])      # 1 to 9 slabs
def test_few_slabs_of_k(gpu_device, K, dtype):
    M, N, g, td = 264, 392, torch.Generator(device="cuda").manual_seed(97), TD[dtype]
    print(f"[case] few slabs K={K} dtype={dtype}", flush=True)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda").to(td)
    nan = lambda *s: torch.full(s, float("nan"), dtype=td, device="cuda")
    x, w, wt, xt = rnd(M, K), rnd(K, N), rnd(N, K), rnd(K, M)
    both(lambda i, C: zs.ops.gemm(st(), dtype, 0, 0, M, N, K, x, K, w, N, C, N, 0, None, None, 0, 1, 0, 0, 0, 0, 0, 0, i), nan(M, N))
    both(lambda i, C: zs.ops.gemm(st(), dtype, 0, 1, M, N, K, x, K, wt, K, C, N, 0, None, None, 0, 1, 0, 0, 0, 0, 0, 0, i), nan(M, N))
    both(lambda i, C: zs.ops.gemm(st(), dtype, 1, 0, M, N, K, xt, M, w, N, C, N, 1, None, None, 0, 1, 0, 0, 0, 0, 0, 0, i),
         torch.randn(M, N, generator=g, device="cuda"))


@pytest.mark.parametrize("dtype", [1, 2])
@pytest.mark.parametrize("parts,each,last", [(2, 128, 8), (2, 128, 128), (3, 128, 72), (2, 256, 200), (5, 128, 128)])
def test_few_slabs_in_parts(gpu_device, parts, each, last, dtype):
    M, N, g, td = 136, 264, torch.Generator(device="cuda").manual_seed(101), TD[dtype]
    print(f"[case] few slabs in parts {parts} x {each}, last {last} dtype={dtype}", flush=True)
    rows = [each] * (parts - 1) + [last]
    x, dy = ([torch.randn(r, w, generator=g, device="cuda").to(td) for r in rows] for w in (M, N))
    both(lambda i, C: zs.wgrad_parts(st(), dtype, M, N, each, last, x, M, dy, N, C, N, 1, 0, 0, 0, i), torch.randn(M, N, generator=g, device="cuda"))
