"""16-bit attention on both sides of the sequence lengths at which rows and results begin, or cease, to pass through LDS as whole lines,
against float64, with the gradients' rows further apart than they are long."""
import pytest
import torch

import paper_2507_10392_amd as zs
from test_attention_backward_one_launch import TD, reference

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [1, 2])
@pytest.mark.parametrize("d,S", [(128, s) for s in (1, 31, 32, 33, 64, 65)] + [(112, s) for s in (33, 64, 65, 255, 256)] +
                         [(80, s) for s in (64, 65, 96, 97, 128, 129, 255, 256)] + [(64, s) for s in (33, 64, 65, 96, 97, 129, 256, 1024, 1025)])
def test_both_ways_match_float64(gpu_device, dtype, d, S):
    mb, nh = 2, 3
    print(f"[case] attention as whole lines S={S} d={d} dtype={dtype}", flush=True)
    g, td, T, H = torch.Generator(device="cuda").manual_seed(89), TD[dtype], mb * S, nh * d
    st = torch.cuda.current_stream().cuda_stream
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda").to(td)
    qkv, do = rnd(T, 3 * H), rnd(T, H)
    o, wide = torch.full((T, H + 8), float("nan"), dtype=td, device="cuda"), torch.full((T + 1, 3 * H + 8), 7.0, dtype=td, device="cuda")
    o, dqkv = o[:, :H], wide[:T, :3 * H]
    dout = torch.empty_strided(o.shape, o.stride(), dtype=td, device="cuda")
    dout.copy_(do)
    lse, delta = torch.empty(mb, nh, S, device="cuda"), torch.empty(mb, nh, S, device="cuda")
    (q, k, v), (dq, dk, dv) = ([a[:, i * H:(i + 1) * H] for i in range(3)] for a in (qkv, dqkv))
    zs.ops.attention_fwd(st, dtype, mb, S, nh, d, q, k, v, 3 * H, o, H + 8, lse, 0)
    zs.ops.attention_bwd(st, dtype, mb, S, nh, d, q, k, v, 3 * H, o, dout, H + 8, lse, delta, dq, dk, dv, 3 * H + 8, 0)
    torch.cuda.synchronize()
    assert (wide[:, 3 * H:] == 7).all() and (wide[T:] == 7).all()          # nothing between the rows or behind them
    # the bounds of the backward's other tests: 16-bit weights and dS, roundings of the results
    tol = {1: 1e-2, 2: 1.25e-3}[dtype]
    for b in range(mb):
        for h in range(nh):
            at = lambda t: t[b * S:(b + 1) * S, h * d:(h + 1) * d]
            z = (at(q).double() @ at(k).double().t() / d ** 0.5).masked_fill(torch.ones(S, S, dtype=torch.bool, device="cuda").triu(1), float("-inf"))
            want = [torch.softmax(z, -1) @ at(v).double(), *reference(at(q), at(k), at(v), at(do))]
            for name, got, ref in zip(("o", "dq", "dk", "dv"), (o, dq, dk, dv), want):
                if S == 1 and name in ("dq", "dk"):                         # exactly zero by a cancellation of dP - delta
                    assert at(got).double().abs().max() <= tol
                    continue
                e = float((at(got).double() - ref).norm() / ref.norm())
                assert e <= tol, f"{name} of head {h}, sequence {b}: {e:.2e}"
