"""Attention gradients that take the place of o (dq, dk or dv) or of k and v, or lie between the columns of one matrix: few row
blocks, where dQ and dK/dV otherwise share a launch.  They have to be those of buffers of their own."""
import pytest
import torch

import paper_2507_10392_amd as zs

pytestmark = pytest.mark.gpu
TD = {0: torch.float32, 1: torch.bfloat16, 2: torch.float16}
TOL = {0: 0.0, 1: 2.0 ** -8, 2: 2.0 ** -11}      # 16 bits: delta is added up in another order, so that a value may round the other way


@pytest.mark.parametrize("dtype,mb,S,nh,d", [(0, 1, 100, 3, 64), (0, 1, 512, 8, 128), (1, 1, 256, 4, 128), (1, 2, 700, 8, 128), (2, 1, 129, 48, 128)])
@pytest.mark.parametrize("place", ["dq over o", "dk over o", "dv over o", "over k and v", "one matrix"])
def test_gradients_in_place(gpu_device, dtype, mb, S, nh, d, place):
    print(f"[case] attention backward in place dtype={dtype} mb={mb} S={S} heads={nh} d={d} {place}", flush=True)
    g, td, T, H = torch.Generator(device="cuda").manual_seed(103), TD[dtype], mb * S, nh * d
    st = torch.cuda.current_stream().cuda_stream
    whole = torch.randn(T, 6 * H, generator=g, device="cuda").to(td)
    W = 6 * H
    q, k, v = (whole[:, i * H:(i + 1) * H] for i in range(3))
    do, o = torch.randn(T, H, generator=g, device="cuda").to(td), torch.empty(T, H, dtype=td, device="cuda")
    lse, delta = torch.empty(mb, nh, S, device="cuda"), torch.empty(mb, nh, S, device="cuda")
    zs.ops.attention_fwd(st, dtype, mb, S, nh, d, q, k, v, W, o, H, lse, 0)

    def backward(o, ldo, do, grads, ldd):
        zs.ops.attention_bwd(st, dtype, mb, S, nh, d, q, k, v, W, o, do, ldo, lse, delta, *grads, ldd, 0)
        torch.cuda.synchronize()
        return [t.clone() for t in grads]

    nan = lambda cols: torch.full((T, cols), float("nan"), dtype=td, device="cuda")
    want = backward(o, H, do, [nan(H) for _ in range(3)], H)
    if place == "over k and v":
        got = backward(o, H, do, [nan(W)[:, :H], k, v], W)
    elif place == "one matrix":
        got = backward(o, H, do, [whole[:, i * H:(i + 1) * H] for i in (3, 4, 5)], W)
    else:
        at = ("dq", "dk", "dv").index(place[:2])
        got = backward(o, H, do, [o if i == at else nan(H) for i in range(3)], H)
    for name, a, b in zip(("dq", "dk", "dv"), got, want):
        assert torch.isfinite(a).all(), name
        assert float((a.double() - b.double()).norm()) <= TOL[dtype] * float(b.double().norm()), name
