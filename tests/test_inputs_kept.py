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
