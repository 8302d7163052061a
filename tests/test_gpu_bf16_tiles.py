"""bf16 products at sizes that take each tile of the dispatch (256 x 256, 256 x 192, 192 x 256, 256 x 128,
128 x 128, 64 x 128, 64 x 64, and whole rounds with a remainder launch), with remainders of the tiles and of
the reduction stages, through halves of a layer: every layout, and every epilogue the layer uses."""
import pytest
import torch

from paper_2504_03662_amd import inputs as I
from paper_2504_03662_amd.runtime import to_device, to_host
from parity import TOL, check, compare, run_both

pytestmark = pytest.mark.gpu

# hidden, ffn, seq, batch: the products are [T, ffn, hidden], [T, hidden, ffn], [hidden, ffn, T] and their like
SHAPES = [
    (64, 8, 1, 1),            # 64 x 64: one token, one chunk of 8
    (128, 72, 65, 1),         # 64 x 64: one row past a tile
    (768, 1032, 129, 2),      # 64 x 64 and 64 x 128
    (512, 4104, 200, 5),      # 64 x 128 and 128 x 128, ragged both ways
    (2048, 1544, 1999, 2),    # 128 x 128 and 256 x 128
    (3072, 3848, 2001, 1),    # 256 x 192, 192 x 256 and 256 x 128
    (2048, 8200, 2050, 1),    # more large tiles than a round
]


@pytest.mark.parametrize("variant", ["f32 gradients", "bf16 gradients, tanh"])
@pytest.mark.parametrize("hidden,ffn,seq,batch", SHAPES)
def test_bf16_feed_forward_half_on_every_tile(hidden, ffn, seq, batch, variant):
    shape = I.LayerShape(hidden, hidden // 64, ffn, 1, 1, 0, seq, batch, "bf16", gelu_tanh=variant != "f32 gradients")
    params = I.full_params(shape, case=500 + seq, random_affine=True)
    x, dy = I.activations(shape, case=500 + seq)
    gpu, ref, layer = run_both(shape, params, x, dy, "mlp")
    compare(gpu, ref, TOL["bf16"], "mlp")
    # accumulating the same gradients again doubles them (fp32 sums are exact; bf16 ones rounded once more)
    layer.wgrad_bf16 = variant != "f32 gradients"
    if layer.wgrad_bf16:
        for n in ("w_fc1", "w_fc2", "w_qkv", "w_o"):
            layer.grads[n] = layer.grads[n].to(torch.bfloat16)
    layer.backward(to_device(x, "bf16"), to_device(dy, "bf16"), "mlp", accumulate=True)
    torch.cuda.synchronize()
    for n in ("w_fc1", "w_fc2"):
        check("d" + n, to_host(layer.grads[n]), 2 * ref["grads"][n], TOL["bf16"])


@pytest.mark.parametrize("phase,hidden,ffn,seq,batch", [
    ("both", 64, 64, 3, 1), ("both", 768, 768, 100, 2), ("both", 1024, 512, 1000, 2), ("attn", 2048, 8, 2001, 1),
    ("both", 3072, 64, 1500, 2),
])
def test_bf16_attention_products_on_every_tile(phase, hidden, ffn, seq, batch):
    shape = I.LayerShape(hidden, hidden // 64, ffn, 1, 1, 0, seq, batch, "bf16")
    params = I.full_params(shape, case=520 + batch, random_affine=True)
    x, dy = I.activations(shape, case=520 + batch)
    gpu, ref, _ = run_both(shape, params, x, dy, phase, want_partials=(phase == "both"))
    compare(gpu, ref, TOL["bf16"], phase, want_partials=(phase == "both"))
