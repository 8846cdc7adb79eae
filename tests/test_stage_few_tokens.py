"""One layer wide enough, on few enough tokens, that the input gradients' products run as two halves of K side by side."""
import pytest

from harness import TOL, GpuStage, compare_step, oracle_step
from workloads import get_config, make_inputs

pytestmark = pytest.mark.gpu


# Llama: gate|up gradients (two segments of the FFN width); GPT: the FFN's and, with K = 3 * hidden, the QKV projection's;
# 136 tokens leave the last tile row ragged
@pytest.mark.parametrize("name,hidden,heads,ffn,seq", [("C3t", 1024, 8, 4096, 256), ("C3h", 1024, 8, 4096, 136), ("C2t", 1024, 8, 8192, 256),
                                                       ("C2t", 2048, 16, 8192, 136)])
def test_layer_on_few_tokens_against_the_oracle(gpu_device, name, hidden, heads, ffn, seq):
    cfg = get_config(name).with_(layers=1, hidden=hidden, heads=heads, ffn=ffn, seq=seq, num_microbatches=1)
    print(f"[case] few tokens {name} hidden={hidden} ffn={ffn} seq={seq}", flush=True)
    scale = 256.0 if cfg.dtype == 2 else 1.0
    inp = make_inputs(cfg, perturbed=True, num_microbatches=1, dy_scale=scale)
    g = GpuStage(cfg, inp, max_microbatches=1)
    gpu = g.run_microbatches(inp, M=1)
    compare_step(cfg, gpu, oracle_step(cfg, inp, M=1), TOL[cfg.dtype])
    g.stage.close()
