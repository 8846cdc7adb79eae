"""16-bit products on 256x192 and 256x128 tiles, and cut along N, as the rule on sizes picks them (impl = 0): every output has to be
the bits of the 256x256 tile (impl = 3, held against float64 elsewhere), which adds the same products in the same order."""
import pytest
import torch

import paper_2507_10392_amd as zs

pytestmark = pytest.mark.gpu
TD = {1: torch.bfloat16, 2: torch.float16}


def st():
    return torch.cuda.current_stream().cuda_stream


def both(dtype, call, *outs):
    """call(impl, *outs) with impl 0 and 3 from the same start; all outputs equal bit for bit."""
    first = [o.clone() for o in outs]
    call(0, *first)
    call(3, *outs)
    torch.cuda.synchronize()
    for a, b in zip(first, outs):
        assert not torch.isnan(b.float()).any()
        assert torch.equal(a.view(torch.uint8), b.view(torch.uint8))


# Most forms of the first two lie on 256x192 (last tile row 249 high, last column 184 wide), of the next two on 256x128 (249 high, 120 wide),
# the last is cut along N: nine tile rows leave 5 of 261 256x256 tiles over.  K: odd and even numbers of 64-wide slabs, the last one
# partly filled.
SIZES = [(1529, 6904, 200), (1529, 6904, 1096), (2041, 4088, 2056), (513, 8192, 2048), (2304, 7400, 1544)]


@pytest.mark.parametrize("dtype", [1, 2])
@pytest.mark.parametrize("M,N,K", SIZES)
def test_same_bits_as_the_square_tile(gpu_device, M, N, K, dtype):
    print(f"[case] oblong tiles M={M} N={N} K={K} dtype={dtype}", flush=True)
    g, td = torch.Generator(device="cuda").manual_seed(71), TD[dtype]
    rnd = lambda *shape, s=1.0: (torch.randn(shape, generator=g, device="cuda") * s).to(td)
    nan = lambda *shape, t=td: torch.full(shape, float("nan"), dtype=t, device="cuda")
    x, w, wt, bias, res = rnd(M, K), rnd(K, N, s=0.05), rnd(N, K, s=0.05), rnd(N), rnd(M, N)
    both(dtype, lambda i, C: zs.ops.gemm(st(), dtype, 0, 0, M, N, K, x, K, w, N, C, N, 0, bias, res, N, 1, 0, 0, 0, 0, 0, 0, i), nan(M, N))
    both(dtype, lambda i, C: zs.ops.gemm(st(), dtype, 0, 1, M, N, K, x, K, wt, K, C, N, 0, None, None, 0, 1, 0, 0, 0, 0, 0, 0, i), nan(M, N))
    seg = K // 2 // 8 * 8      # two segments of K, whose boundary lies inside a slab
    both(dtype, lambda i, C: zs.ops.gemm(st(), dtype, 0, 1, M, N, 2 * seg, x, K, wt, seg, C, N, 0, None, None, 0, 1, 0, 0, 0, 0, seg, N * seg, i), nan(M, N))
    K8, T = (M + 7) // 8 * 8, K // 8 * 8
    xt, dy = rnd(T, K8), rnd(T, N)
    both(dtype, lambda i, C: zs.ops.gemm(st(), dtype, 1, 0, K8, N, T, xt, K8, dy, N, C, N, 1, None, None, 0, 1, 0, 0, 0, 0, 0, 0, i),
         torch.randn(K8, N, generator=g, device="cuda"))
    F = N // 16 * 8            # gate and up side by side, and the derivative in the store
    wgu = rnd(2, K, F, s=0.05)
    both(dtype, lambda i, a, gu: zs.ops.gemm_glu(st(), dtype, 1, M, F, K, x, K, wgu, F, K * F, a, gu, i), nan(M, F), nan(M, 2 * F))
    scratch = nan(M, N)
    both(dtype, lambda i, gu: zs.ops.gemm_glu(st(), dtype, 2, M, N, K, x, K, wt, K, 0, scratch, gu, i), rnd(M, 2 * N))
    S, d = 24, 8               # the rotation in the store
    table = torch.empty(S, d // 2, 2, device="cuda")
    zs.ops.rope_table(st(), S, d, 10000.0, table)
    both(dtype, lambda i, C: zs.ops.gemm_rope(st(), dtype, 0, 0, M, N, K, x, K, w, N, C, N, 0, None, None, 0, 1, 0, 0, 0, 0, 0, 0, i, table, S, d, 1), nan(M, N))


def forced(dtype, tile, call, *outs):
    """The same with the tile (3: 256x192, 4: 256x128) forced, as the library's own choice would take it, against the 256x256 tile."""
    force = getattr(zs.lib(), "_ZN2zs20gemm_mfma_force_tileEi")      # zs::gemm_mfma_force_tile(int): holds for the next call

    def one(impl, *o):
        if impl == 0:
            force(tile)
            impl = 2
        call(impl, *o)
    both(dtype, one, *outs)


# one tile and a bit of the next each way, or less than one; 1, 2, 3, 4 and 5 slabs of K, the last one partly filled or full
@pytest.mark.parametrize("dtype", [1, 2])
@pytest.mark.parametrize("tile", [3, 4])
@pytest.mark.parametrize("M,N,K", [(8, 16, 8), (249, 120, 72), (257, 200, 128), (512, 392, 136), (520, 136, 256), (264, 584, 264)])
def test_every_form_on_a_forced_oblong_tile(gpu_device, M, N, K, tile, dtype):
    print(f"[case] forced tile {tile} M={M} N={N} K={K} dtype={dtype}", flush=True)
    g, td = torch.Generator(device="cuda").manual_seed(73), TD[dtype]
    rnd = lambda *shape, s=1.0: (torch.randn(shape, generator=g, device="cuda") * s).to(td)
    nan = lambda *shape, t=td: torch.full(shape, float("nan"), dtype=t, device="cuda")
    x, w, wt, bias, res = rnd(M, K), rnd(K, N, s=0.05), rnd(N, K, s=0.05), rnd(N), rnd(M, N)
    forced(dtype, tile, lambda i, C: zs.ops.gemm(st(), dtype, 0, 0, M, N, K, x, K, w, N, C, N, 0, bias, res, N, 1, 0, 0, 0, 0, 0, 0, i), nan(M, N))
    forced(dtype, tile, lambda i, C: zs.ops.gemm(st(), dtype, 0, 1, M, N, K, x, K, wt, K, C, N, 0, None, None, 0, 1, 0, 0, 0, 0, 0, 0, i), nan(M, N))
    forced(dtype, tile, lambda i, C: zs.ops.gemm(st(), dtype, 0, 1, M, N, K, x, K, wt, K, C, N, 1, None, None, 0, 1, 0, 0, 0, 0, 0, 0, i),
           torch.randn(M, N, generator=g, device="cuda"))      # x W^T added to fp32
    if K % 16 == 0:
        forced(dtype, tile, lambda i, C: zs.ops.gemm(st(), dtype, 0, 1, M, N, K, x, K, wt, K // 2, C, N, 0, None, None, 0, 1, 0, 0, 0, 0, K // 2,
                                                     N * K // 2, i), nan(M, N))
    M8 = (M + 7) // 8 * 8
    xt, dy = rnd(2, K, M8), rnd(2, K, N)
    forced(dtype, tile, lambda i, C: zs.ops.gemm(st(), dtype, 1, 0, M8, N, K, xt, M8, dy, N, C, N, 1, None, None, 0, 2, K * M8, K * N, M8 * N, 0, 0, 0, i),
           torch.randn(2, M8, N, generator=g, device="cuda"))
    F = max(N // 16 * 8, 8)
    wgu, scratch = rnd(2, K, F, s=0.05), nan(M, N)
    forced(dtype, tile, lambda i, a, gu: zs.ops.gemm_glu(st(), dtype, 1, M, F, K, x, K, wgu, F, K * F, a, gu, i), nan(M, F), nan(M, 2 * F))
    forced(dtype, tile, lambda i, gu: zs.ops.gemm_glu(st(), dtype, 2, M, N, K, x, K, wt, K, 0, scratch, gu, i), rnd(M, 2 * N))
