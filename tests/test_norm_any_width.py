"""Norms over rows of any width: masked last vectors, rows shared by two, four and eight waves, rows too long for registers."""
import numpy as np
import pytest
import torch

import paper_2507_10392_amd as zs
from harness import dev, log_report, rel_err
from workloads import round_bf16, round_f16

pytestmark = pytest.mark.gpu
TD = {0: torch.float32, 1: torch.bfloat16, 2: torch.float16}
TOL = {0: 2e-5, 1: 1e-2, 2: 1.5e-3}      # the bars of the other single-kernel tests: one rounding of the outputs
EPS = 1e-5


@pytest.mark.parametrize("dtype", [0, 1, 2])
@pytest.mark.parametrize("kind", [0, 1])
# widths in chunks of 64 lanes x 16 bytes (256 fp32 or 512 16-bit elements).  Backward: within the first and 2 and a bit, one wave
# per row; 5 and a bit (three chunks per wave) and 7 and a bit (four), two waves; just over 8 (three per wave) and just under 16,
# four waves; just over 16 and 32, eight waves; just over 32, re-reading kernels.  Forward: one wave up to 16, then re-reading.
@pytest.mark.parametrize("chunks,T,nblk", [(0.125, 5, 5), (2.0625, 37, 7), (5.0625, 21, 5), (5.5, 10, 3), (7.5, 33, 4), (8.0625, 19, 6),
                                           (15.9375, 9, 2), (16.0625, 11, 3), (32, 6, 6), (32.0625, 3, 2)])
def test_norm_any_width(gpu_device, kind, dtype, chunks, T, nblk):
    H = int(chunks * (256 if dtype == 0 else 512))
    print(f"[case] norm kind={kind} dtype={dtype} T={T} H={H} nblk={nblk}", flush=True)
    rng = np.random.default_rng(71)
    td = TD[dtype]
    rnd = {0: lambda a: a, 1: round_bf16, 2: round_f16}[dtype]
    f = lambda *s, scale=1.0, base=0.0: rnd((base + scale * rng.standard_normal(s)).astype(np.float32))
    x, g, b, dn, dres = f(T, H, scale=2.0), f(H, base=1.0, scale=0.1), f(H, scale=0.1), f(T, H), f(T, H)
    x64, g64, b64, dn64 = (a.astype(np.float64) for a in (x, g, b, dn))
    mu = x64.mean(1, keepdims=True) if kind == 0 else np.zeros((T, 1))
    r = 1 / np.sqrt(((x64 - mu) ** 2).mean(1, keepdims=True) + EPS)
    xhat = (x64 - mu) * r
    u = dn64 * g64
    dx = r * (u - (u.mean(1, keepdims=True) if kind == 0 else 0) - xhat * (u * xhat).mean(1, keepdims=True)) + dres
    per = -(-T // nblk)
    block = lambda a: np.stack([a[i * per:(i + 1) * per].sum(0) for i in range(nblk)])
    want = {"n": xhat * g64 + (b64 if kind == 0 else 0), "rstd": r[:, 0], "dx": dx, "dg": block(dn64 * xhat)}
    nan = lambda *s, dt=torch.float32: torch.full(s, float("nan"), dtype=dt, device="cuda")
    got = {"n": nan(T, H, dt=td), "rstd": nan(T), "dx": dev(dres, td), "dg": nan(nblk, H)}
    mean, db = (nan(T), nan(nblk, H)) if kind == 0 else (None, None)
    st = torch.cuda.current_stream().cuda_stream
    xd, gd, bd, dnd = dev(x, td), dev(g, td), dev(b, td) if kind == 0 else None, dev(dn, td)
    zs.ops.norm_fwd(st, dtype, kind, T, H, xd, gd, bd, EPS, got["n"], got["rstd"], mean)
    # dres aliases dx, as in the stage
    zs.ops.norm_bwd(st, dtype, kind, T, H, dnd, xd, gd, got["rstd"], mean, got["dx"], got["dx"], got["dg"], db, nblk)
    if kind == 0:
        want.update(mean=mu[:, 0], db=block(dn64))
        got.update(mean=mean, db=db)
    torch.cuda.synchronize()
    errs = [(n, rel_err(got[n].float().cpu().numpy(), want[n])) for n in want]
    log_report(f"norm {kind} {dtype} {T} {H}", errs)
    for n, e in errs:
        assert e <= (TOL[dtype] if n in ("n", "dx") else 2e-5), n
