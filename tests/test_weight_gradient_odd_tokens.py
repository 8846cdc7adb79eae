"""16-bit weight gradients over a number of tokens that is no multiple of 8, on the matrix cores (impl = 0)."""
import numpy as np
import pytest
import torch

import paper_2507_10392_amd as zs
from harness import dev, log_report, rel_err
from workloads import round_bf16, round_f16

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [1, 2])
@pytest.mark.parametrize("M,N,T,batch", [(8, 8, 1, 1), (136, 264, 7, 2), (264, 136, 65, 1), (520, 1376, 1021, 3), (2048, 2056, 127, 1)])
def test_weight_gradient_over_an_odd_number_of_tokens(gpu_device, dtype, M, N, T, batch):
    print(f"[case] wgrad M={M} N={N} T={T} batch={batch} dtype={dtype}", flush=True)
    rng = np.random.default_rng(51)
    rnd, td = (round_bf16, torch.bfloat16) if dtype == 1 else (round_f16, torch.float16)
    # rows behind the last token hold inf: nothing past it may be read into the sums
    x, dy = (rnd(rng.standard_normal((T + 9, w)).astype(np.float32)) for w in (M, batch * N))
    x[T:], dy[T:] = np.inf, np.inf
    C0 = rng.standard_normal((batch, M, N)).astype(np.float32)
    C = dev(C0)
    zs.ops.gemm(torch.cuda.current_stream().cuda_stream, dtype, 1, 0, M, N, T, dev(x, td), M, dev(dy, td), batch * N, C, N, 1, None, None, 0,
                batch, 0, N, M * N, 0, 0, 0, 0)
    torch.cuda.synchronize()
    want = np.stack([C0[z] + x[:T].astype(np.float64).T @ dy[:T, z * N:(z + 1) * N].astype(np.float64) for z in range(batch)])
    err = rel_err(C.cpu().numpy(), want)
    log_report(f"odd wgrad {M} {N} {T} {batch} {dtype}", [("C", err)])
    assert err <= 2e-5            # exact 16-bit products, fp32 sums: the bar of the other accumulating products


@pytest.mark.parametrize("dtype", [1, 2])
# 32x32 and 64x64 tiles, then staged tiles
@pytest.mark.parametrize("M,N,parts,last", [(40, 72, 3, 1), (520, 1376, 2, 77), (1000, 1016, 5, 127), (2048, 2056, 3, 77), (2048, 4104, 4, 201)])
def test_last_of_several_parts_with_an_odd_number_of_tokens(gpu_device, M, N, parts, last, dtype):
    print(f"[case] wgrad parts M={M} N={N} parts={parts} last={last} dtype={dtype}", flush=True)
    rng = np.random.default_rng(52)
    rnd, td = (round_bf16, torch.bfloat16) if dtype == 1 else (round_f16, torch.float16)
    rows = [128] * (parts - 1) + [last]
    x, dy = ([rnd(rng.standard_normal((r + 9, w)).astype(np.float32)) for r in rows] for w in (M, N))
    for a, b, r in zip(x, dy, rows):     # rows behind a part's last token hold inf
        a[r:], b[r:] = np.inf, np.inf
    C0 = rng.standard_normal((M, N)).astype(np.float32)
    C = dev(C0)
    zs.wgrad_parts(torch.cuda.current_stream().cuda_stream, dtype, M, N, 128, last, [dev(a, td) for a in x], M, [dev(a, td) for a in dy], N, C, N,
                   1, 0, 0, 0, 0)
    torch.cuda.synchronize()
    want = C0 + sum(a[:r].astype(np.float64).T @ b[:r].astype(np.float64) for a, b, r in zip(x, dy, rows))
    err = rel_err(C.cpu().numpy(), want)
    log_report(f"odd wgrad parts {M} {N} {parts} {last} {dtype}", [("C", err)])
    assert err <= 2e-5            # exact 16-bit products, fp32 sums: the bar of the other accumulating products


@pytest.mark.parametrize("M,N,T,ld", [(64, 64, 3, 72 * 2 ** 20), (4096, 4096, 31, 33 * 2 ** 19), (64, 64, 3, 2 ** 27)])
def test_rows_so_far_apart_that_the_tile_would_wrap_around(gpu_device, M, N, T, ld):
    """A tile's k-lines past the last token, at 32-bit byte offsets beyond 2^32, must not come back into the operand."""
    print(f"[case] wgrad with far rows M={M} N={N} T={T} ld={ld}", flush=True)
    torch.manual_seed(53)
    x, dy = (torch.randn(T * ld, device="cuda", dtype=torch.bfloat16) for _ in range(2))
    C = torch.zeros(M, N, device="cuda")
    zs.ops.gemm(torch.cuda.current_stream().cuda_stream, 1, 1, 0, M, N, T, x, ld, dy, ld, C, N, 1, None, None, 0, 1, 0, 0, 0, 0, 0, 0, 0)
    torch.cuda.synchronize()
    a, b = (t.view(T, ld)[:, :w].double().cpu().numpy() for t, w in ((x, M), (dy, N)))
    assert rel_err(C.cpu().numpy(), a.T @ b) <= 2e-5


def test_forced_matrix_core_kernel_still_wants_multiples_of_8(gpu_device):
    x, dy, C = (torch.zeros(64, 64, device="cuda", dtype=t) for t in (torch.bfloat16, torch.bfloat16, torch.float32))
    with pytest.raises(zs.StageError):
        zs.ops.gemm(torch.cuda.current_stream().cuda_stream, 1, 1, 0, 64, 64, 63, x, 64, dy, 64, C, 64, 1, None, None, 0, 1, 0, 0, 0, 0, 0, 0, 2)
