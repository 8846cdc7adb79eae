"""Attention where single tokens hold inf or NaN: a token that a row does not see must not reach it, and the rows that do see it
get what the wave-per-row kernel (impl = 1), which skips masked keys, gives them."""
import numpy as np
import pytest
import torch

import paper_2507_10392_amd as zs
from harness import dev

pytestmark = pytest.mark.gpu
TD = {0: torch.float32, 1: torch.bfloat16, 2: torch.float16}
# largest difference of two correct results over the largest value: fp32 sums in another order, or two roundings of the output
BAR = {0: 5e-6, 1: 2.0 ** -7, 2: 2.0 ** -10}


def st():
    return torch.cuda.current_stream().cuda_stream


def forward(dtype, mb, S, nh, d, qkv, impl):
    H = nh * d
    q, k, v = (qkv[:, i * H:(i + 1) * H] for i in range(3))
    o = torch.full((mb * S, H), 7.0, dtype=TD[dtype], device="cuda")
    lse = torch.full((mb, nh, S), 7.0, device="cuda")
    zs.ops.attention_fwd(st(), dtype, mb, S, nh, d, q, k, v, 3 * H, o, H, lse, impl)
    return o, lse


def backward(dtype, mb, S, nh, d, qkv, o, do, lse, impl, rope=None):
    H = nh * d
    q, k, v = (qkv[:, i * H:(i + 1) * H] for i in range(3))
    dqkv = torch.full((mb * S, 3 * H), 7.0, dtype=TD[dtype], device="cuda")
    delta = torch.empty(mb * nh * S, device="cuda")
    zs.ops.attention_bwd_rope(st(), dtype, mb, S, nh, d, q, k, v, 3 * H, o, do, H, lse, delta, dqkv[:, :H], dqkv[:, H:2 * H],
                              dqkv[:, 2 * H:], 3 * H, impl, rope)
    return dqkv


def same(name, got, want, bar):
    torch.cuda.synchronize()
    g, w = (t.float().cpu().numpy().astype(np.float64) for t in (got, want))
    assert (np.isnan(g) == np.isnan(w)).all(), f"{name}: NaN at {np.argwhere(np.isnan(g) != np.isnan(w))[:4].tolist()}"
    assert (np.isinf(g) == np.isinf(w)).all() and (g[np.isinf(g)] == w[np.isinf(w)]).all(), f"{name}: inf"
    f = np.isfinite(w)
    assert not f.any() or np.abs(g[f] - w[f]).max() <= bar * np.abs(w[f]).max(), name


# one block; a last block of one row; several tiles and, in 16 bits above S = 256, rows that two waves share; padded head dims.  fp32: dQ and
# dK/dV in one launch up to 256 blocks of 16 rows, in two above (25 heads)
CASES = [(0, 1, 45, 2, 64), (0, 2, 97, 1, 40), (0, 1, 161, 1, 128), (0, 1, 161, 25, 128), (0, 1, 170, 25, 40),
         *((t, *c) for t in (1, 2) for c in ((1, 45, 2, 64), (2, 97, 1, 40), (1, 300, 2, 64), (1, 161, 1, 96), (1, 321, 1, 104)))]


@pytest.mark.parametrize("dtype,mb,S,nh,d", CASES)
@pytest.mark.parametrize("bad", [float("inf"), float("-inf"), float("nan")])
def test_a_value_row_reaches_only_the_queries_that_see_it(gpu_device, dtype, mb, S, nh, d, bad):
    print(f"[case] non-finite V dtype={dtype} mb={mb} S={S} nh={nh} d={d} {bad}", flush=True)
    rng = np.random.default_rng(61)
    H = nh * d
    x = rng.standard_normal((mb * S, 3 * H)).astype(np.float32)
    for row, col in ((S - 1, 3), (S // 2 + 3, d - 1), (S // 2, 0)):
        x[row, 2 * H + col] = bad
    qkv = dev(x, TD[dtype])
    (o, lse), (want, want_lse) = (forward(dtype, mb, S, nh, d, qkv, i) for i in (0, 1))
    same("o", o, want, BAR[dtype])
    same("lse", lse, want_lse, 5e-6)
    assert torch.isfinite(o[:S // 2]).all()


@pytest.mark.parametrize("dtype,mb,S,nh,d", CASES)
@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
@pytest.mark.parametrize("which", ["q", "k", "do"])
@pytest.mark.parametrize("rotate", [False, True])
def test_gradients_of_the_rows_that_do_not_see_it_stay_finite(gpu_device, dtype, mb, S, nh, d, bad, which, rotate):
    """k: queries before the row keep their dq.  q, do: keys behind the row keep their dk and dv."""
    print(f"[case] non-finite {which} dtype={dtype} mb={mb} S={S} nh={nh} d={d} {bad} rotate={rotate}", flush=True)
    rng = np.random.default_rng(62)
    H, row = nh * d, S // 2 + 1
    x, y = (rng.standard_normal((mb * S, w)).astype(np.float32) for w in (3 * H, H))
    {"q": x, "k": x[:, H:], "do": y}[which][row, 5] = bad
    qkv, do = dev(x, TD[dtype]), dev(y, TD[dtype])
    o, lse = forward(dtype, mb, S, nh, d, qkv, 1)
    table = None
    if rotate:
        table = torch.empty(S, d // 2, 2, device="cuda")
        zs.ops.rope_table(st(), S, d, 10000.0, table)
    got, want = (backward(dtype, mb, S, nh, d, qkv, o, do, lse, i, table) for i in (0, 1))
    for n, at in (("dq", 0), ("dk", 1), ("dv", 2)):
        same(n, got[:, at * H:(at + 1) * H], want[:, at * H:(at + 1) * H], 2 * BAR[dtype])
    clean = got[:row, :H] if which == "k" else got[row + 1:S, H:]
    assert torch.isfinite(clean).all()


@pytest.mark.parametrize("mb,S,nh,d", [(1, 45, 2, 64), (1, 300, 2, 64), (1, 161, 1, 96), (1, 70, 1, 104)])
def test_half_gradients_beyond_the_range_of_the_split(gpu_device, mb, S, nh, d):
    """dS above 2^20, where its high half part overflows, with Q and K so small that dq and dk are ordinary half values."""
    print(f"[case] large dS mb={mb} S={S} nh={nh} d={d}", flush=True)
    rng = np.random.default_rng(63)
    H = nh * d
    x = rng.standard_normal((mb * S, 3 * H)).astype(np.float32)
    x[:, :2 * H] *= 1e-3
    x[:, 2 * H:] *= 300.0
    do = dev((1e4 * np.clip(rng.standard_normal((mb * S, H)), -2, 2)).astype(np.float32), TD[2])
    qkv = dev(x, TD[2])
    o, lse = forward(2, mb, S, nh, d, qkv, 0)
    v, g = qkv[:, 2 * H:].double(), do.double()
    ds = (v * g).view(mb * S, nh, d)[1].sum(-1) / 2     # two keys, probabilities of about a half: dS of the second query's own
    assert ds.abs().max() > 2.0 ** 20 and torch.isfinite(o).all()
    got, want = (backward(2, mb, S, nh, d, qkv, o, do, lse, i) for i in (0, 1))
    assert torch.isfinite(want).all()
    for n, at in (("dq", 0), ("dk", 1), ("dv", 2)):
        same(n, got[:, at * H:(at + 1) * H], want[:, at * H:(at + 1) * H], BAR[2])
