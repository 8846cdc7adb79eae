"""The weight gradients of a layer that share one launch (gemm_group), at the edges of their tiles, against the fp64 oracle."""
import pytest

from harness import TOL, GpuStage, compare_step, oracle_step
from workloads import get_config, make_inputs

pytestmark = pytest.mark.gpu

# (config, changes): tiles are 32x64 (fp32) or 64x64 (16 bits), slabs of K 16 or 32 rows shared by 8 (fp32; 4 from 2049 tiles on) or 2 waves
CASES = [
    ("C1", dict(layers=1, seq=1, microbatch=1)),                                            # one row of K
    ("C1", dict(layers=1, hidden=72, heads=3, ffn=104, seq=13, microbatch=1)),              # ragged in M, N and K, waves without a slab
    ("C1", dict(layers=2, hidden=264, heads=3, ffn=1032, seq=67, microbatch=2)),            # two layers write gradients of their own
    ("L1", dict(layers=1, hidden=144, heads=2, ffn=200, seq=65, microbatch=1)),             # batches of two and three
    ("C1", dict(layers=1, hidden=1088, heads=17, ffn=3000, seq=65, microbatch=1)),          # 5000 tiles
    ("C2h", dict(layers=1, hidden=64, heads=1, ffn=136, seq=64, microbatch=1)),             # one column of tiles
    ("C3t", dict(layers=1, seq=31, microbatch=1)),                                          # less than a slab
    ("C3t", dict(layers=2, hidden=264, heads=3, ffn=1000, seq=77, microbatch=1)),
    ("C3h", dict(layers=1, hidden=520, heads=5, ffn=1384, seq=225, microbatch=2)),
]


@pytest.mark.parametrize("name,changes", CASES)
def test_grouped_weight_gradients_match_the_oracle(gpu_device, name, changes):
    cfg = get_config(name).with_(num_microbatches=2, **changes)
    print(f"[case] grouped weight gradients {name} {changes}", flush=True)
    inp = make_inputs(cfg, perturbed=True, num_microbatches=2)
    g = GpuStage(cfg, inp, max_microbatches=2)
    g.stage.profile(True)
    gpu = g.run_microbatches(inp, M=2)      # the second microbatch is added to the first one's gradients
    rows = g.stage.profile_read()
    g.stage.close()
    per_layer = 2 * cfg.layers
    tn = {k: v["launches"] for k, v in rows.items() if "_tn" in k}
    assert sum(tn.values()) == per_layer + (2 if cfg.has_head else 0), tn
    compare_step(cfg, gpu, oracle_step(cfg, inp, M=2), TOL[cfg.dtype])


# fp32 layers whose products fill their rounds of 128x128 tiles keep them: grouped, on smaller tiles, they are slower
@pytest.mark.parametrize("seq,launches", [(256, 1), (640, 4)])
def test_fp32_layers_that_fill_their_rounds_are_not_grouped(gpu_device, seq, launches):
    cfg = get_config("C1").with_(layers=1, hidden=2048, heads=16, ffn=8192, seq=seq, microbatch=1, num_microbatches=1)
    print(f"[case] fp32 weight gradients, hidden 2048, {seq} tokens", flush=True)
    inp = make_inputs(cfg, perturbed=True, num_microbatches=1)
    g = GpuStage(cfg, inp, max_microbatches=1)
    g.stage.profile(True)
    gpu = g.run_microbatches(inp, M=1)
    rows = g.stage.profile_read()
    g.stage.close()
    assert rows["gemm_f32_tn"]["launches"] == launches, rows
    compare_step(cfg, gpu, oracle_step(cfg, inp, M=1), TOL[cfg.dtype])
