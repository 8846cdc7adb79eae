"""16-bit attention with head dims below 128 on the matrix cores (impl = 0) against the oracle and against the
wave-per-row fp32 kernel (impl = 1), whose precision it keeps."""
import numpy as np
import pytest
import torch

import paper_2507_10392_amd as zs
from harness import dev, log_report, rel_err
from oracle import stage_oracle as so
from workloads import round_bf16, round_f16

pytestmark = pytest.mark.gpu
TD = {1: torch.bfloat16, 2: torch.float16}


def st():
    return torch.cuda.current_stream().cuda_stream


def back(t):
    torch.cuda.synchronize()
    return t.float().cpu().numpy().astype(np.float64)


def run(dtype, mb, S, nh, d, qkv, do, impl, rope=None, shift=0):
    """shift: elements by which the rows start off a 16-byte boundary."""
    H, td = nh * d, TD[dtype]
    ld = 3 * H + 8
    buf = torch.zeros(mb * S * ld + 8, dtype=td, device="cuda")
    x = torch.as_strided(buf, (mb * S, 3 * H), (ld, 1), shift)
    x.copy_(dev(qkv, td))
    q, k, v = (x[:, i * H:(i + 1) * H] for i in range(3))
    o = torch.full((mb * S, H), float("nan"), dtype=td, device="cuda")
    lse = torch.full((mb, nh, S), float("nan"), device="cuda")
    dqkv = torch.full((mb * S, 3 * H), float("nan"), dtype=td, device="cuda")
    delta = torch.empty(mb * nh * S, device="cuda")
    zs.ops.attention_fwd(st(), dtype, mb, S, nh, d, q, k, v, ld, o, H, lse, impl)
    zs.ops.attention_bwd_rope(st(), dtype, mb, S, nh, d, q, k, v, ld, o, dev(do, td), H, lse, delta, dqkv[:, :H], dqkv[:, H:2 * H],
                              dqkv[:, 2 * H:], 3 * H, impl, rope)
    return {"o": back(o), "lse": back(lse), "dq": back(dqkv[:, :H]), "dk": back(dqkv[:, H:2 * H]), "dv": back(dqkv[:, 2 * H:])}


def rms(a, b):
    return np.sqrt(np.mean((a - b) ** 2) / max(np.mean(b ** 2), 1e-300))


@pytest.mark.parametrize("dtype", [1, 2])
@pytest.mark.parametrize("mb,S,nh,d", [(1, 1, 1, 8), (2, 63, 3, 40), (1, 65, 2, 64), (2, 200, 3, 64), (1, 129, 2, 72), (2, 130, 2, 96),
                                       (1, 257, 1, 104), (1, 70, 2, 120)])
def test_narrow_heads_match_the_oracle_as_closely_as_fp32(gpu_device, mb, S, nh, d, dtype):
    print(f"[case] attention mb={mb} S={S} nh={nh} d={d} dtype={dtype}", flush=True)
    rng = np.random.default_rng(41)
    rnd = round_bf16 if dtype == 1 else round_f16
    H = nh * d
    qkv, do = (rnd(rng.standard_normal((mb * S, w)).astype(np.float32)) for w in (3 * H, H))
    q, k, v = (qkv[:, i * H:(i + 1) * H].astype(np.float64).reshape(mb, S, nh, d) for i in range(3))
    g = so.attention_bwd(do.astype(np.float64).reshape(mb, S, nh, d), q, k, v)
    want = {"o": so.attention_fwd(q, k, v).reshape(mb * S, H), **{n: a.reshape(mb * S, H) for n, a in zip(("dq", "dk", "dv"), g)}}
    s = np.einsum("bihd,bjhd->bhij", q, k) / np.sqrt(d)
    s = np.where(np.tril(np.ones((S, S), bool)), s, -np.inf)
    want["lse"] = np.log(np.exp(s).sum(-1))
    got, plain = run(dtype, mb, S, nh, d, qkv, do, 0), run(dtype, mb, S, nh, d, qkv, do, 1)
    log_report(f"narrow attention {mb} {S} {nh} {d} {dtype}", [(n, rel_err(got[n], want[n])) for n in want])
    for n in want:
        if not np.abs(want[n]).max() > 1e-12:     # one key: its probability does not depend on q and k
            assert np.abs(got[n]).max() <= 1e-3
            continue
        # the rounding of the outputs dominates both: their errors differ by the luck of single roundings only
        assert rms(got[n], want[n]) <= 1.05 * rms(plain[n], want[n]) + 3e-8, n


@pytest.mark.parametrize("dtype", [1, 2])
def test_keys_that_hardly_any_query_sees_keep_their_gradients(gpu_device, dtype):
    """Probabilities of 1e-6 and smaller: dk and dv of such keys are as good as the fp32 kernel's, relative to themselves."""
    mb, S, nh, d = 1, 192, 2, 64
    print(f"[case] small probabilities dtype={dtype}", flush=True)
    rng = np.random.default_rng(42)
    rnd = round_bf16 if dtype == 1 else round_f16
    H = nh * d
    qkv = rng.standard_normal((S, 3 * H)).astype(np.float32)
    qkv[:, :H] = 1.0 + 0.1 * qkv[:, :H]
    qkv[64::2, H:2 * H] -= 1.75       # every second key from 64 on: scores lower by about 14
    qkv, do = rnd(qkv), rnd(rng.standard_normal((S, H)).astype(np.float32) * 100)
    got, plain = run(dtype, mb, S, nh, d, qkv, do, 0), run(dtype, mb, S, nh, d, qkv, do, 1)
    q, k, v = (qkv[:, i * H:(i + 1) * H].astype(np.float64).reshape(mb, S, nh, d) for i in range(3))
    g = so.attention_bwd(do.astype(np.float64).reshape(mb, S, nh, d), q, k, v)
    for n, a in zip(("dq", "dk", "dv"), g):
        a = a.reshape(S, H)[66:190:2]
        assert rms(got[n][66:190:2], a) <= 1.1 * rms(plain[n][66:190:2], a) + 1e-6, n


@pytest.mark.parametrize("dtype", [1, 2])
def test_narrow_heads_with_inverse_rotation_and_unaligned_rows(gpu_device, dtype):
    mb, S, nh, d = 2, 75, 2, 80
    print(f"[case] narrow attention, rotation, unaligned rows dtype={dtype}", flush=True)
    rng = np.random.default_rng(43)
    rnd = round_bf16 if dtype == 1 else round_f16
    H = nh * d
    qkv, do = (rnd(rng.standard_normal((mb * S, w)).astype(np.float32)) for w in (3 * H, H))
    table = torch.empty(S, d // 2, 2, device="cuda")
    zs.ops.rope_table(st(), S, d, 10000.0, table)
    plain = run(dtype, mb, S, nh, d, qkv, do, 1, table)
    unit = 2.0 ** (-8 if dtype == 1 else -11)
    for shift in (0, 4):              # 4: the wave-per-row kernel takes it
        got = run(dtype, mb, S, nh, d, qkv, do, 0, table, shift)
        for n in plain:               # impl 1 rounds dq and dk once more, before it rotates them: two roundings apart at most
            assert rel_err(got[n], plain[n]) <= 2 * unit, (n, shift)


@pytest.mark.parametrize("dtype", [1, 2])
@pytest.mark.parametrize("mb,S,nh", [(1, 31, 1), (2, 257, 1), (1, 321, 2), (1, 384, 3), (1, 385, 3)])
def test_heads_of_128_whose_rows_two_waves_share(gpu_device, mb, S, nh, dtype):
    """Backward of few head-sequences (8 waves per block of 128 rows, two on the same 32) against the oracle; the last block
    holds 1, 31, 65 or 128 rows."""
    d = 128
    print(f"[case] attention bwd mb={mb} S={S} nh={nh} dtype={dtype}", flush=True)
    rng = np.random.default_rng(44)
    rnd = round_bf16 if dtype == 1 else round_f16
    H = nh * d
    qkv, do = (rnd(rng.standard_normal((mb * S, w)).astype(np.float32)) for w in (3 * H, H))
    q, k, v = (qkv[:, i * H:(i + 1) * H].astype(np.float64).reshape(mb, S, nh, d) for i in range(3))
    g = so.attention_bwd(do.astype(np.float64).reshape(mb, S, nh, d), q, k, v)
    got = run(dtype, mb, S, nh, d, qkv, do, 0)
    for n, a in zip(("dq", "dk", "dv"), g):
        # probabilities and dS are rounded to 16 bits, as before, then the sums: the bar of the other 16-bit attention tests
        assert rel_err(got[n], a.reshape(mb * S, H)) <= 2e-2, n
