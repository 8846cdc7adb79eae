"""A stage keeps what it needs of a microbatch's inputs: the caller may reuse the buffers once the forward has run."""
import numpy as np
import pytest
import torch

from harness import GpuStage, dev, tdtype
from workloads import get_config, make_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("seq,recompute", [(256, 0), (131, 0), (131, 1)])
def test_inputs_overwritten_after_the_forward(gpu_device, seq, recompute):
    cfg = get_config("C5t").with_(seq=seq, num_microbatches=2, recompute=recompute)
    print(f"[case] inputs kept seq={seq} recompute={recompute}", flush=True)
    inp = make_inputs(cfg, num_microbatches=2)
    grads, outs = [], []
    for overwrite in (False, True):
        g = GpuStage(cfg, inp, max_microbatches=2)
        ys, bufs = [], []
        for i in range(2):
            ids, tg = dev(inp.ids[i].reshape(-1)), dev(inp.targets[i].reshape(-1))
            y = torch.full((cfg.tokens, cfg.hidden), 7.0, dtype=tdtype(cfg), device="cuda")
            loss = torch.zeros(1, device="cuda")
            g.stage.forward(i, ids, y, tg, loss)
            ys.append(y.clone())
            if overwrite:
                ids.zero_(); tg.zero_(); y.zero_()
            bufs.append((ids, tg, y, loss))
        for i in (1, 0):
            g.stage.backward(i, None, None, 0.5)
            g.stage.accumulate(i)
        torch.cuda.synchronize()
        grads.append(g.grad.cpu().numpy().copy())
        outs.append([y.float().cpu().numpy() for y in ys] + [b[3].item() for b in bufs])
        g.stage.close()
    assert np.array_equal(grads[0], grads[1]) and np.any(grads[0])
    for a, b in zip(*outs):
        assert np.array_equal(a, b) and np.all(a != 7.0)


@pytest.mark.parametrize("name", ["C1", "C3t", "C2h"])
@pytest.mark.parametrize("recompute", [0, 1])
def test_stage_input_overwritten_after_the_forward(gpu_device, name, recompute):
    """A stage in the middle of a pipeline, which takes activations: the input buffer zeroed after the forward, the output written
    over the input, and an input that starts one element off its 16-byte boundary give the bits of the ordinary call."""
    cfg = get_config(name).with_(layers=2, seq=131, num_microbatches=1, recompute=recompute)
    inp = make_inputs(cfg, num_microbatches=1)
    want = None
    for how in ("plain", "zeroed", "in place", "unaligned"):
        print(f"[case] stage input {how} {name} recompute={recompute}", flush=True)
        g = GpuStage(cfg, inp, max_microbatches=1)
        td, shape = tdtype(cfg), (cfg.tokens, cfg.hidden)
        x = dev(inp.x[0], td).reshape(shape)
        if how == "unaligned":
            x = torch.empty(x.numel() + 8, dtype=td, device="cuda")[1:x.numel() + 1].view(shape).copy_(x)
            assert x.data_ptr() % 16
        y = x if how == "in place" else torch.full(shape, 7.0, dtype=td, device="cuda")
        g.stage.forward(0, x, y, None, None)
        out = y.clone()
        if how in ("zeroed", "in place"):
            x.zero_()
        dx = torch.full(shape, 7.0, dtype=td, device="cuda")
        g.stage.backward(0, dev(inp.dy[0], td), dx, 1.0)
        g.stage.accumulate(0)
        torch.cuda.synchronize()
        got = [t.float().cpu().numpy() for t in (out, dx, g.grad)]
        g.stage.close()
        want = want or got
        assert np.any(got[2]) and all(np.array_equal(a, b) for a, b in zip(got, want)), how
