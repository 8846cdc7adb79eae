"""Layers on few tokens, whose input gradients have few tiles and a long K, against the oracle."""
import pytest

from harness import TOL, GpuStage, compare_step, oracle_step
from workloads import get_config, make_inputs

pytestmark = pytest.mark.gpu


def run(name, hidden, heads, ffn, seq, M=1, **more):
    cfg = get_config(name).with_(**{"layers": 1, **more}, hidden=hidden, heads=heads, ffn=ffn, seq=seq, num_microbatches=M)
    print(f"[case] few tokens {name} hidden={hidden} ffn={ffn} seq={seq} {more}", flush=True)
    scale = 256.0 if cfg.dtype == 2 else 1.0
    inp = make_inputs(cfg, perturbed=True, num_microbatches=M, dy_scale=scale)
    g = GpuStage(cfg, inp, max_microbatches=M)
    g.stage.profile(True)
    gpu = g.run_microbatches(inp, M=M)
    classes = g.stage.profile_read()
    compare_step(cfg, gpu, oracle_step(cfg, inp, M=M), TOL[cfg.dtype])
    g.stage.close()
    return classes


# small enough for the 32x32 tiles of gemm_small.hip, K in two segments (Llama) and in one (GPT); 136 tokens leave the last tile
# row ragged
@pytest.mark.parametrize("name,hidden,heads,ffn,seq", [("C3t", 1024, 8, 4096, 256), ("C3h", 1024, 8, 4096, 136), ("C2t", 1024, 8, 8192, 256),
                                                       ("C2t", 2048, 16, 8192, 136)])
def test_layer_on_few_tokens_against_the_oracle(gpu_device, name, hidden, heads, ffn, seq):
    assert "gemm_small_nt" in run(name, hidden, heads, ffn, seq)


# 80 tiles of 128x128: too many for the small tiles, and so few that the two halves of K run side by side as fp32 results in
# scratch.  Llama: the gate|up gradient (its two segments become the batch); GPT: the FFN's and, where the scratch that is free at
# its time holds two results (ffn >= 4 hidden), the QKV projection's.  600 tokens leave the last tile row ragged.
@pytest.mark.parametrize("name,ffn,seq,products", [("C3t", 2048, 640, 1), ("C3t", 2056, 600, 1), ("C3h", 2048, 600, 1), ("C2t", 8192, 600, 2),
                                                   ("C2h", 8192, 640, 2), ("C2h", 4096, 600, 1)])
def test_input_gradients_as_two_halves_of_k(gpu_device, name, ffn, seq, products):
    classes = run(name, 2048, 16, ffn, seq)
    assert classes.get("gemm_halves_nt", {"launches": 0})["launches"] == products, sorted(classes)


# Llama with ffn >= 2 hidden: the QKV projection's three segments run as a batch of three, whose results lie over the microbatch's
# saved gate, up and activation; the last size's batch is on 256x128 tiles, the others' on 128x128.
@pytest.mark.parametrize("name,hidden,heads,ffn,seq", [("C3t", 2048, 16, 5120, 640), ("C3h", 2048, 16, 6144, 600), ("C3t", 4096, 32, 8192, 320)])
def test_input_gradient_as_three_segments(gpu_device, name, hidden, heads, ffn, seq):
    assert run(name, hidden, heads, ffn, seq)["gemm_parts_nt"]["launches"] == 1


# pair_wgrad, three backwards: the first one's weight gradients wait, so it keeps what they read and its QKV gradient runs in one part;
# the second multiplies for both, the third for itself.  Recomputation: the layer's saved values are made again for each microbatch.
@pytest.mark.parametrize("more,M,launches", [(dict(pair_wgrad=1), 3, 2), (dict(recompute=1, layers=2), 2, 4)])
def test_three_segments_over_several_microbatches(gpu_device, more, M, launches):
    assert run("C3t", 2048, 16, 5120, 640, M, **more)["gemm_parts_nt"]["launches"] == launches


@pytest.mark.parametrize("name,vocab", [("C5t", 8000), ("C5h", 8016)])
def test_lm_head_gradient_as_two_halves(gpu_device, name, vocab):
    """The scratch lies over buffers that the layers' backward writes later.  The FFN's gradient is the other product in halves."""
    assert run(name, 2048, 16, 2048, 640, vocab=vocab)["gemm_halves_nt"]["launches"] == 2


# Forward products of 80 or 96 tiles in two microbatches: the FFN's down projection, with its residual (GPT: and bias), and where K is long
# enough the attention output's, in two halves over scratch of the backward, also beside gradients (recomputation, of two layers, makes the
# attention output again for each, and not the down projection, whose result nothing reads).
@pytest.mark.parametrize("name,hidden,heads,ffn,seq,more,launches", [
    ("C3t", 2048, 16, 5120, 640, {}, 4), ("C3h", 2048, 16, 5136, 600, {}, 4), ("C2t", 2048, 16, 8192, 600, {}, 4), ("C2h", 2048, 16, 8192, 760, {}, 2),
    ("C3t", 4096, 32, 8192, 320, {}, 4), ("C2t", 4096, 32, 8192, 300, {}, 4), ("C3t", 2048, 16, 8192, 640, dict(recompute=1, layers=2), 12),
    ("C3h", 4096, 32, 8192, 320, dict(recompute=1, layers=2), 12)])
def test_forward_products_as_two_halves_of_k(gpu_device, name, hidden, heads, ffn, seq, more, launches):
    assert run(name, hidden, heads, ffn, seq, 2, **more)["gemm_halves_nn"]["launches"] == launches
