"""fp32 GPT layers, whose GELU and its derivative are part of the FFN products' stores where the fp32 matrix cores take those, against the
oracle: 16x16 to 64x64 tiles with ragged edges."""
import pytest

from harness import TOL, GpuStage, compare_step, oracle_step
from workloads import get_config, make_inputs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hidden,heads,ffn,seq,mb", [(32, 2, 40, 3, 1), (72, 3, 104, 19, 1), (128, 2, 1032, 77, 2), (256, 4, 2056, 300, 2)])
@pytest.mark.parametrize("recompute", [0, 1])
def test_gelu_of_fp32_layers(gpu_device, hidden, heads, ffn, seq, mb, recompute):
    cfg = get_config("C1").with_(layers=2, hidden=hidden, heads=heads, ffn=ffn, seq=seq, microbatch=mb, num_microbatches=2, recompute=recompute)
    print(f"[case] GELU in the store hidden={hidden} ffn={ffn} seq={seq} mb={mb} recompute={recompute}", flush=True)
    inp = make_inputs(cfg, perturbed=True, num_microbatches=2)
    g = GpuStage(cfg, inp, max_microbatches=2)
    g.stage.profile(True)
    gpu = g.run_microbatches(inp, M=2)
    classes = g.stage.profile_read()
    compare_step(cfg, gpu, oracle_step(cfg, inp, M=2), TOL[cfg.dtype])
    g.stage.close()
    assert "activation" not in classes, sorted(classes)
