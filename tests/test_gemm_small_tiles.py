"""16-bit products with outputs too small for the staged tiles (impl = 0), at the edges of 32x32 and 64x64 tiles, against
float64; every form that a stage uses."""
import numpy as np
import pytest
import torch

import paper_2507_10392_amd as zs
from harness import dev, log_report, rel_err
from workloads import round_bf16, round_f16

pytestmark = pytest.mark.gpu
TD = {1: torch.bfloat16, 2: torch.float16}
UNIT = {1: 2.0 ** -8, 2: 2.0 ** -11}     # a rounding to the 16-bit type, relative


def st():
    return torch.cuda.current_stream().cuda_stream


def draw(rng, shape, dtype, scale=1.0):
    a = (rng.standard_normal(shape) * scale).astype(np.float32)
    return round_bf16(a) if dtype == 1 else round_f16(a)


def back(t):
    torch.cuda.synchronize()
    return t.float().cpu().numpy().astype(np.float64)


# fewer than 8 slabs of 32 k (idle waves), K that ends inside one, one output tile, ragged tiles; the last two take 64x64
SIZES = [(1, 8, 8), (31, 40, 72), (33, 64, 264), (256, 520, 1000), (100, 264, 2752), (1000, 1016, 520), (1030, 1000, 1032)]


@pytest.mark.parametrize("dtype", [1, 2])
@pytest.mark.parametrize("M,N,K", SIZES)
def test_forward_and_input_gradient_forms(gpu_device, M, N, K, dtype):
    print(f"[case] small gemm M={M} N={N} K={K} dtype={dtype}", flush=True)
    rng = np.random.default_rng(61)
    td, batch = TD[dtype], 2
    A, B, bias, R = draw(rng, (M, K), dtype), draw(rng, (batch, K, N), dtype, 0.05), draw(rng, (batch, N), dtype), draw(rng, (batch, M, N), dtype)
    want = A.astype(np.float64) @ B.astype(np.float64) + bias[:, None] + R
    C = torch.full((batch, M, N), float("nan"), dtype=td, device="cuda")
    zs.ops.gemm(st(), dtype, 0, 0, M, N, K, dev(A, td), K, dev(B, td), N, C, N, 0, dev(bias, td), dev(R, td), N, batch, 0, K * N, M * N, N, 0,
                0, 0)
    errs = [("nn", rel_err(back(C), want))]
    staged = torch.empty_like(C)     # the forward form sums in the order of the staged kernels
    zs.ops.gemm(st(), dtype, 0, 0, M, N, K, dev(A, td), K, dev(B, td), N, staged, N, 0, dev(bias, td), dev(R, td), N, batch, 0, K * N, M * N, N,
                0, 0, 2)
    torch.cuda.synchronize()
    assert torch.equal(C.view(torch.int16), staged.view(torch.int16))
    # the same weights stored [N, K], whole and in segments of K along the contraction
    want = A.astype(np.float64) @ B[0].astype(np.float64)
    C = torch.full((M, N), float("nan"), dtype=td, device="cuda")
    zs.ops.gemm(st(), dtype, 0, 1, M, N, K, dev(A, td), K, dev(np.ascontiguousarray(B[0].T), td), K, C, N, 0, None, None, 0, 1, 0, 0, 0, 0, 0, 0, 0)
    errs.append(("nt", rel_err(back(C), want)))
    A2 = draw(rng, (M, 2 * K), dtype)
    want = A2[:, :K].astype(np.float64) @ B[0].astype(np.float64) + A2[:, K:].astype(np.float64) @ B[1].astype(np.float64)
    segs = np.ascontiguousarray(B.transpose(0, 2, 1))
    C = torch.full((M, N), float("nan"), dtype=td, device="cuda")
    zs.ops.gemm(st(), dtype, 0, 1, M, N, 2 * K, dev(A2, td), 2 * K, dev(segs, td), K, C, N, 0, None, None, 0, 1, 0, 0, 0, 0, K, N * K, 0)
    errs.append(("segments", rel_err(back(C), want)))
    log_report(f"small gemm {M} {N} {K} {dtype}", errs)
    for n, e in errs:      # one rounding of the largest value, and fp32 sums of K terms well below it
        assert e <= UNIT[dtype], n


@pytest.mark.parametrize("dtype", [1, 2])
@pytest.mark.parametrize("M,N,T,parts", [(8, 8, 128, 2), (40, 72, 128, 3), (520, 1376, 256, 1), (1000, 1016, 128, 5)])
def test_weight_gradient_of_several_parts(gpu_device, M, N, T, parts, dtype):
    print(f"[case] small wgrad M={M} N={N} T={T} parts={parts} dtype={dtype}", flush=True)
    rng = np.random.default_rng(62)
    td, last, batch = TD[dtype], T // 2 + 8, 2
    rows = [T] * (parts - 1) + [last]
    x, dy = ([draw(rng, (r, w), dtype) for r in rows] for w in (M, batch * N))
    C0 = rng.standard_normal((batch, M, N)).astype(np.float32)
    C = dev(C0)
    zs.wgrad_parts(st(), dtype, M, N, T, last, [dev(a, td) for a in x], M, [dev(a, td) for a in dy], batch * N, C, N, batch, 0, N, M * N, 0)
    want = np.stack([C0[z] + sum(a.astype(np.float64).T @ b[:, z * N:(z + 1) * N].astype(np.float64) for a, b in zip(x, dy)) for z in range(batch)])
    err = rel_err(back(C), want)
    log_report(f"small wgrad {M} {N} {T} {parts} {dtype}", [("C", err)])
    assert err <= 2e-5     # exact products, fp32 sums: the bar of the other accumulating products


@pytest.mark.parametrize("dtype", [1, 2])
@pytest.mark.parametrize("M,N,K", [(40, 72, 136), (256, 1376, 512), (500, 1000, 264)])
def test_gated_unit_and_rotation_in_the_store(gpu_device, M, N, K, dtype):
    """Backward of the gated unit against its formulas; gate and up fused against the batched product, bit for bit; the
    rotated projection against the plain one followed by the oracle's rotation."""
    print(f"[case] small gemm, fused stores M={M} N={N} K={K} dtype={dtype}", flush=True)
    rng = np.random.default_rng(63)
    td = TD[dtype]
    x, w = dev(draw(rng, (M, K), dtype), td), dev(draw(rng, (2, K, N), dtype, 0.05), td)
    a, gu, a2, gu2 = (torch.full((M, c), float("nan"), dtype=td, device="cuda") for c in (N, 2 * N, N, 2 * N))
    zs.ops.gemm_glu(st(), dtype, 1, M, N, K, x, K, w, N, K * N, a, gu, 0)
    zs.ops.gemm(st(), dtype, 0, 0, M, N, K, x, K, w, N, gu2, 2 * N, 0, None, None, 0, 2, 0, K * N, N, 0, 0, 0, 0)
    zs.ops.swiglu(st(), dtype, M, N, gu2, None, a2, 0)
    assert torch.equal(gu, gu2) and torch.equal(a, a2)
    dy, wd = draw(rng, (M, K), dtype), draw(rng, (N, K), dtype, 0.05)
    da = dy.astype(np.float64) @ wd.astype(np.float64).T
    gv, uv = back(gu)[:, :N], back(gu)[:, N:]
    sg = 1 / (1 + np.exp(-gv))
    want = np.concatenate([da * uv * sg * (1 + gv * (1 - sg)), da * gv * sg], 1)
    zs.ops.gemm_glu(st(), dtype, 2, M, N, K, dev(dy, td), K, dev(wd, td), K, 0, a, gu, 0)
    assert rel_err(back(gu), want) <= UNIT[dtype]
    S, d = 20, 8
    table = torch.empty(S, d // 2, 2, device="cuda")
    zs.ops.rope_table(st(), S, d, 10000.0, table)
    plain, got = (torch.full((M, 2 * N), float("nan"), dtype=td, device="cuda") for _ in range(2))
    zs.ops.gemm_rope(st(), dtype, 0, 0, M, N, K, x, K, w, N, got, 2 * N, 0, None, None, 0, 2, 0, K * N, N, 0, 0, 0, 0, table, S, d, 1)
    p = (back(x) @ back(w[0])).reshape(M, N // 2, 2)
    t = back(table)
    cs, sn = (np.tile(t[np.arange(M) % S, :, i], (1, N // d)) for i in range(2))
    want = np.stack([p[..., 0] * cs - p[..., 1] * sn, p[..., 0] * sn + p[..., 1] * cs], -1).reshape(M, N)
    assert rel_err(back(got)[:, :N], want) <= UNIT[dtype]
    assert rel_err(back(got)[:, N:], back(x) @ back(w[1])) <= UNIT[dtype]
