"""The attention backward whose dQ and dK/dV share a launch (few row blocks; in 16 bits heads of 128 only), at the edges of its
rules and of its tiles, against float64."""
import pytest
import torch

import paper_2507_10392_amd as zs

pytestmark = pytest.mark.gpu
D = 128
TD = {1: torch.bfloat16, 2: torch.float16}
# (mb, S, heads): the last sizes that share a launch and the first that do not, for one, two and more blocks of 128 rows per head
SIZES = [(1, 1, 3), (1, 63, 2), (2, 65, 2), (1, 127, 128), (1, 128, 129), (2, 129, 48), (1, 256, 97), (3, 257, 16), (1, 700, 42), (1, 700, 43)]


def reference(q, k, v, do):
    """Gradients of one head in float64."""
    q, k, v = (t.double().requires_grad_() for t in (q, k, v))
    S = q.shape[0]
    z = (q @ k.t() / q.shape[1] ** 0.5).masked_fill(torch.ones(S, S, dtype=torch.bool, device=q.device).triu(1), float("-inf"))
    o = torch.softmax(z, -1) @ v
    o.backward(do.double())
    return q.grad, k.grad, v.grad


@pytest.mark.parametrize("dtype", [1, 2])
@pytest.mark.parametrize("mb,S,nh", SIZES)
def test_gradients_match_float64(gpu_device, mb, S, nh, dtype):
    print(f"[case] attention backward in one launch mb={mb} S={S} heads={nh} dtype={dtype}", flush=True)
    g, td, T, H = torch.Generator(device="cuda").manual_seed(83), TD[dtype], mb * S, nh * D
    st = torch.cuda.current_stream().cuda_stream
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda").to(td)
    qkv, do = rnd(T, 3 * H), rnd(T, H)
    o, dqkv = torch.empty_like(do), torch.full_like(qkv, float("nan"))
    lse, delta = torch.empty(mb, nh, S, device="cuda"), torch.full((mb, nh, S), float("nan"), device="cuda")
    q, k, v = (qkv[:, i * H:(i + 1) * H] for i in range(3))
    dq, dk, dv = (dqkv[:, i * H:(i + 1) * H] for i in range(3))
    zs.ops.attention_fwd(st, dtype, mb, S, nh, D, q, k, v, 3 * H, o, H, lse, 0)
    zs.ops.attention_bwd(st, dtype, mb, S, nh, D, q, k, v, 3 * H, o, do, H, lse, delta, dq, dk, dv, 3 * H, 0)
    torch.cuda.synchronize()
    assert torch.isfinite(dqkv).all()
    want = (do.double() * o.double()).reshape(mb, S, nh, D).sum(-1).permute(0, 2, 1)
    assert (delta.double() - want).abs().max() <= 1e-5 * want.abs().max()      # 128 fp32 additions: 128 * 2^-24
    # 16-bit weights and dS (a rounding of 2^-9 or 2^-12 each, whose signs are independent) and the rounded O behind delta
    tol = {1: 1e-2, 2: 1.25e-3}[dtype]
    for b, h in {(0, 0), (mb - 1, nh - 1), (mb // 2, nh // 2)}:
        at = lambda t: t[b * S:(b + 1) * S, h * D:(h + 1) * D]
        for name, got, ref in zip(("dq", "dk", "dv"), (dq, dk, dv), reference(at(q), at(k), at(v), at(do))):
            if S == 1 and name != "dv":                                         # exactly zero by a cancellation of dP - delta
                assert at(got).double().abs().max() <= tol
                continue
            e = float((at(got).double() - ref).norm() / ref.norm())
            assert e <= tol, f"{name} of head {h}, sequence {b}: {e:.2e}"


def backward_f32(qkv, do, mb, S, nh, d):
    H, st = nh * d, torch.cuda.current_stream().cuda_stream
    o, dqkv = torch.empty_like(do), torch.full_like(qkv, float("nan"))
    lse, delta = torch.empty(mb, nh, S, device="cuda"), torch.full((mb, nh, S), float("nan"), device="cuda")
    q, k, v = (qkv[:, i * H:(i + 1) * H] for i in range(3))
    dq, dk, dv = (dqkv[:, i * H:(i + 1) * H] for i in range(3))
    zs.ops.attention_fwd(st, 0, mb, S, nh, d, q, k, v, 3 * H, o, H, lse, 0)
    zs.ops.attention_bwd(st, 0, mb, S, nh, d, q, k, v, 3 * H, o, do, H, lse, delta, dq, dk, dv, 3 * H, 0)
    torch.cuda.synchronize()
    return dqkv.reshape(mb * S, 3, nh, d), delta


# blocks have 16 rows; tiles 32; S * heads up to 256 blocks
@pytest.mark.parametrize("mb,S,nh,d", [(1, 33, 2, 128), (2, 47, 3, 64), (1, 100, 3, 80), (1, 129, 28, 40), (1, 512, 8, 128)])
@pytest.mark.parametrize("infinite", [False, True])
def test_fp32_same_bits_as_separate_launches(gpu_device, mb, S, nh, d, infinite):
    """The same heads among enough others for separate launches.  infinite: a value whose products overflow, so that rows are redone."""
    print(f"[case] fp32 attention backward in one launch mb={mb} S={S} heads={nh} d={d} infinite={infinite}", flush=True)
    g, T, times = torch.Generator(device="cuda").manual_seed(89), mb * S, 256 // (mb * -(-S // 16) * nh) + 1
    qkv, do = torch.randn(T, 3, nh, d, generator=g, device="cuda"), torch.randn(T, nh, d, generator=g, device="cuda")
    if infinite:
        do[S // 2, nh - 1, d // 2] = 3e38
        qkv[S // 3, 2, nh - 1, d // 2] = 1e30
    grad, delta = backward_f32(qkv.reshape(T, -1), do.reshape(T, -1), mb, S, nh, d)
    more, more_delta = backward_f32(qkv.repeat(1, 1, times, 1).reshape(T, -1), do.repeat(1, times, 1).reshape(T, -1), mb, S, nh * times, d)
    clean = nh - 1 if infinite else nh      # a redone row adds delta up in another order
    assert torch.equal(grad[:, :, :clean], more[:, :, :clean]) and torch.equal(delta[:, :clean], more_delta[:, :clean])
    assert torch.equal(grad.isfinite(), more[:, :, :nh].isfinite())
    if infinite:      # two orders of d fp32 additions per delta: d * 2^-23 of its terms, which the largest finite gradient is made of
        for a, b in zip(grad[:, :, nh - 1].unbind(1), more[:, :, nh - 1].unbind(1)):
            f = a.isfinite()
            assert (a[f].double() - b[f].double()).abs().max() <= d * 2.0 ** -23 * b[f].double().abs().max()
        return
    for got, ref in zip(grad[:S, :, 0].unbind(1), reference(*qkv[:S, :, 0].unbind(1), do[:S, 0])):
        assert float((got.double() - ref).norm() / ref.norm()) <= 2e-5
