"""stage_profile_read names the kernels that the dispatch chose."""
import pytest

from harness import GpuStage
from workloads import get_config, make_inputs

pytestmark = pytest.mark.gpu


# (config, changes, classes that must appear, prefixes that must not)
CASES = [
    ("L1", {}, {"gemm_f32_nn", "gemm_f32_nt", "gemm_f32_tn", "attn_fwd_f32", "attn_bwd_f32"}, ("gemm_simple", "gemm_small", "attn_fwd_simple")),
    ("L1", dict(hidden=272, heads=2), {"gemm_f32_nn", "attn_fwd_simple", "attn_bwd_simple"}, ("attn_fwd_f32", "attn_bwd_f32")),
    # too few keys for the matrix cores: a wave per row (with heads of 64, in bf16 in the forward only)
    ("C1", dict(seq=4), {"attn_fwd_simple", "attn_bwd_simple"}, ("attn_fwd_f32", "attn_bwd_f32")),
    ("L1", dict(seq=4), {"attn_fwd_simple", "attn_bwd_f32"}, ("attn_fwd_f32", "attn_bwd_simple")),     # rotated gradients
    ("C3t", dict(heads=8, seq=4), {"attn_fwd_simple", "attn_bwd_mfma_split"}, ("attn_fwd_mfma_split",)),
    ("C3t", dict(heads=8), {"gemm_small_nn", "gemm_small_tn", "gemm_small_nn_glu", "attn_fwd_mfma_split", "attn_bwd_mfma_split"},
     ("gemm_f32", "gemm_simple", "attn_fwd_simple")),
    ("C3h", {}, {"gemm_small_nn", "attn_fwd_mfma", "attn_bwd_mfma"}, ("gemm_f32", "attn_fwd_mfma_split")),
    # weight gradients over few tokens have many small tiles with hardly any K: staged tiles
    ("C3t", dict(hidden=2048, heads=16, ffn=2048, seq=48), {"gemm_mfma_tn"}, ("gemm_small_tn",)),
    ("C3t", dict(hidden=1024, heads=8, ffn=4096, seq=2048), {"gemm_mfma_nn", "gemm_mfma_nt", "gemm_mfma_tn", "gemm_mfma_nn_glu"}, ("gemm_simple",)),
]


@pytest.mark.parametrize("name,changes,present,absent", CASES)
def test_classes_name_the_kernels_that_ran(gpu_device, name, changes, present, absent):
    cfg = get_config(name).with_(layers=1, num_microbatches=1, **changes)
    print(f"[case] timing classes {name} {changes}", flush=True)
    inp = make_inputs(cfg, num_microbatches=1)
    g = GpuStage(cfg, inp, max_microbatches=1)
    g.stage.profile(True)
    g.run_microbatches(inp, M=1)
    got = set(g.stage.profile_read())
    g.stage.close()
    assert present <= got, present - got
    assert not [n for n in got if n.startswith(absent)], got
