"""The fp32 matrix-core kernels (what impl = 0 runs in the fp32 configuration) at the edges of their tiles, against float64."""
import numpy as np
import pytest
import torch

import paper_2507_10392_amd as zs
from harness import dev, log_report, rel_err
from oracle import stage_oracle as so

pytestmark = pytest.mark.gpu


def st():
    return torch.cuda.current_stream().cuda_stream


def back(t):
    torch.cuda.synchronize()
    return t.cpu().numpy().astype(np.float64)


GEMM_CASES = [
    # (M, N, K, transA, transB, batch, kseg, bias, resid, accum)
    (4, 4, 4, 0, 1, 1, 0, True, True, False),             # one quad of outputs
    (1, 4, 20, 0, 0, 1, 0, False, False, False),
    (31, 36, 132, 0, 0, 2, 0, True, True, False),         # 16x16 tiles, ragged
    (252, 260, 100, 1, 0, 1, 0, False, False, True),      # 16x32, both operands row-contiguous
    (100, 132, 52, 1, 0, 1, 0, True, False, False),       # 16x16, both operands row-contiguous
    (256, 260, 688, 0, 1, 3, 0, True, False, False),      # 32x32
    (260, 64, 1, 1, 0, 1, 0, False, False, True),         # one row of K
    (36, 1376, 77, 1, 0, 3, 0, True, True, True),         # odd K, accumulating with bias and residual
    (520, 1000, 203, 1, 0, 2, 0, False, False, True),     # 64x64 tiles
    (68, 72, 52, 1, 1, 1, 0, False, False, False),
    (130, 68, 5 * 12, 0, 1, 1, 12, False, False, False),  # segments shorter than a slab
    (257, 512, 2 * 344, 0, 1, 1, 344, False, False, False),
    (1100, 2052, 260, 0, 0, 2, 0, True, True, False),     # 64x64, several rounds of workgroups
    (1028, 2052, 131, 1, 0, 2, 0, False, False, True),
    # 128x128 tiles, ragged, in every form: 765 workgroups are three rounds of the 256 CUs and 2970 of 64x64 twelve, by the rule's
    # estimate half as long again
    (1100, 2052, 68, 0, 0, 5, 0, True, True, False),
    (1100, 2052, 68, 0, 1, 5, 0, False, False, False),
    (1100, 2052, 72, 0, 1, 5, 36, True, False, False),
    (1028, 2052, 67, 1, 0, 5, 0, False, False, True),
    (1028, 2052, 68, 1, 1, 5, 0, False, True, False),
    (130, 70, 50, 0, 0, 1, 0, True, True, False),         # contiguous extents that are no multiples of 4: the plain kernel
]


@pytest.mark.parametrize("case", GEMM_CASES, ids=lambda c: "x".join(str(int(v)) for v in c))
def test_gemm_f32_matches_float64(gpu_device, case):
    M, N, K, ta, tb, batch, kseg, use_bias, use_res, accum = case
    print(f"[case] gemm f32 {case}", flush=True)
    rng = np.random.default_rng(31)
    f = lambda *s: rng.standard_normal(s).astype(np.float32)
    A = f(batch, K, M) if ta else f(batch, M, K)
    nseg = K // kseg if kseg else 1
    B = f(nseg, N, kseg) if kseg else f(batch, N, K) if tb else f(batch, K, N)
    bias, R, C0 = f(batch, N), f(batch, M, N), f(batch, M, N)
    want = np.empty((batch, M, N))
    for z in range(batch):
        a = A[z].astype(np.float64).T if ta else A[z].astype(np.float64)
        b = (np.concatenate([B[s].astype(np.float64).T for s in range(nseg)], axis=0) if kseg
             else B[z].astype(np.float64).T if tb else B[z].astype(np.float64))
        want[z] = a @ b + use_bias * bias[z][None, :] + use_res * R[z].astype(np.float64) + accum * C0[z]
    dC = dev(C0) if accum else torch.full((batch, M, N), float("nan"), device="cuda")
    dA, dB, dbias, dR = dev(A), dev(B), dev(bias) if use_bias else None, dev(R) if use_res else None
    zs.ops.gemm(st(), 0, ta, tb, M, N, K, dA, M if ta else K, dB, (kseg or K) if tb else N, dC, N, int(accum), dbias, dR, N, batch,
                M * K, 0 if kseg else N * K, M * N, N, kseg, N * kseg if kseg else 0, 0)
    err = rel_err(back(dC), want)
    log_report(f"gemm f32 {case}", [("C", err)])
    # K roundings of at most half an ulp (6e-8) of partial sums that grow like sqrt(k): 6e-8 * sqrt(K) of the largest sum
    # is 2e-6 at K = 1376; the bar of the other fp32 kernels is ten times that
    assert err <= 2e-5


def test_gemm_f32_rotation_in_the_store(gpu_device):
    """Q|K|V projection as a batch of three whose first two results are rotated: as the plain product followed by
    stage_op_rope, to fp32 rounding."""
    mb, S, nh, d = 2, 37, 3, 40
    T, H = mb * S, nh * d
    print("[case] gemm f32 + rope", flush=True)
    rng = np.random.default_rng(32)
    x, w = dev(rng.standard_normal((T, H)).astype(np.float32)), dev(rng.standard_normal((3, H, H)).astype(np.float32))
    table = torch.empty(S, d // 2, 2, device="cuda")
    zs.ops.rope_table(st(), S, d, 10000.0, table)
    got, want = (torch.full((T, 3 * H), float("nan"), device="cuda") for _ in range(2))
    zs.ops.gemm_rope(st(), 0, 0, 0, T, H, H, x, H, w, H, got, 3 * H, 0, None, None, 0, 3, 0, H * H, H, 0, 0, 0, 0, table, S, d, 2)
    zs.ops.gemm(st(), 0, 0, 0, T, H, H, x, H, w, H, want, 3 * H, 0, None, None, 0, 3, 0, H * H, H, 0, 0, 0, 1)
    scratch = torch.empty(S, d // 2, 2, device="cuda")
    zs.ops.rope(st(), 0, T, S, 2 * H, d, want, 3 * H, 10000.0, 1.0, scratch)
    assert rel_err(back(got), back(want)) <= 2e-6


def attention(mb, S, nh, d, qkv, do, impl, table=None, shift=0):
    """shift: elements by which the rows start off a 16-byte boundary."""
    H = nh * d
    ld = 3 * H + 4
    x = torch.as_strided(torch.zeros(mb * S * ld + 8, device="cuda"), (mb * S, 3 * H), (ld, 1), shift)
    x.copy_(dev(qkv))
    q, k, v = (x[:, i * H:(i + 1) * H] for i in range(3))
    o, dqkv = (torch.full((mb * S, w), float("nan"), device="cuda") for w in (H, 3 * H))
    lse, delta = torch.full((mb, nh, S), float("nan"), device="cuda"), torch.empty(mb, nh, S, device="cuda")
    zs.ops.attention_fwd(st(), 0, mb, S, nh, d, q, k, v, ld, o, H, lse, impl)
    zs.ops.attention_bwd_rope(st(), 0, mb, S, nh, d, q, k, v, ld, o, dev(do), H, lse, delta, dqkv[:, :H], dqkv[:, H:2 * H],
                              dqkv[:, 2 * H:], 3 * H, impl, table)
    return {"o": back(o), "lse": back(lse), "dq": back(dqkv[:, :H]), "dk": back(dqkv[:, H:2 * H]), "dv": back(dqkv[:, 2 * H:])}


# one row; ends inside a 16-row block, on it and past it; more tiles of 32 rows than waves; head dims that fill 16-, 64- and
# 128-column pieces partly; 136 and the unaligned rows below run on the wave-per-row kernel
@pytest.mark.parametrize("mb,S,nh,d", [(1, 1, 1, 8), (2, 15, 1, 24), (1, 16, 3, 64), (2, 33, 2, 40), (1, 161, 2, 64), (2, 130, 1, 72),
                                       (1, 97, 2, 128), (1, 20, 1, 136)])
def test_attention_f32_matches_the_oracle(gpu_device, mb, S, nh, d):
    print(f"[case] attention f32 mb={mb} S={S} nh={nh} d={d}", flush=True)
    rng = np.random.default_rng(33)
    H = nh * d
    qkv, do = (rng.standard_normal((mb * S, w)).astype(np.float32) for w in (3 * H, H))
    q, k, v = (qkv[:, i * H:(i + 1) * H].astype(np.float64).reshape(mb, S, nh, d) for i in range(3))
    g = so.attention_bwd(do.astype(np.float64).reshape(mb, S, nh, d), q, k, v)
    want = {"o": so.attention_fwd(q, k, v).reshape(mb * S, H), **{n: a.reshape(mb * S, H) for n, a in zip(("dq", "dk", "dv"), g)}}
    s = np.einsum("bihd,bjhd->bhij", q, k) / np.sqrt(d)
    want["lse"] = np.log(np.exp(np.where(np.tril(np.ones((S, S), bool)), s, -np.inf)).sum(-1))
    got = attention(mb, S, nh, d, qkv, do, 0)
    for n in want:
        if S == 1 and n in ("dq", "dk"):      # one key: its probability does not depend on q and k
            assert np.abs(got[n]).max() <= 1e-5
            continue
        err = rel_err(got[n], want[n])
        log_report(f"attention f32 {mb} {S} {nh} {d}", [(n, err)])
        assert err <= (2e-5 if n in ("o", "lse") else 5e-5), n      # the bars of the other fp32 attention tests


def test_attention_f32_rotation_and_unaligned_rows(gpu_device):
    mb, S, nh, d = 2, 45, 2, 40
    print("[case] attention f32, rotation, unaligned rows", flush=True)
    rng = np.random.default_rng(34)
    qkv, do = (rng.standard_normal((mb * S, w * nh * d)).astype(np.float32) for w in (3, 1))
    table = torch.empty(S, d // 2, 2, device="cuda")
    zs.ops.rope_table(st(), S, d, 10000.0, table)
    want = attention(mb, S, nh, d, qkv, do, 1, table)
    for shift in (0, 1):                      # 1: the wave-per-row kernel takes it
        got = attention(mb, S, nh, d, qkv, do, 0, table, shift)
        for n in want:
            assert rel_err(got[n], want[n]) <= 5e-6, (n, shift)
