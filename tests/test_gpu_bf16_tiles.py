"""bf16 products through layers and halves of layers.  First, with shapes that the launcher's own rule is
asked about: every layout and epilogue that the layer uses on each tile that it can take there, in its steady
loop, with the four forms of a weight gradient (fp32 or bf16, stored or added to).  Then ragged and tiny sizes:
remainders of the tiles and of the reduction stages, products shorter than the stages in flight."""
import pytest
import torch

from paper_2504_03662_amd import inputs as I
from paper_2504_03662_amd.runtime import to_device, to_host
from bf16_tiles import SHAPES as EVERY_KERNEL
from parity import TOL, check, compare, run_both

pytestmark = pytest.mark.gpu

WEIGHTS = ("w_qkv", "w_o", "w_fc1", "w_fc2")


@pytest.mark.parametrize("phase,shape", EVERY_KERNEL, ids=[f"{p}-{s.hidden}-{s.hidden_local}-{s.ffn}-{s.seq}" for p, s in EVERY_KERNEL])
def test_bf16_every_product_kernel(phase, shape):
    params = I.rank_params(shape, case=540, random_affine=True)
    x, dy = I.activations(shape, case=540)
    gpu, ref, layer = run_both(shape, params, x, dy, phase)
    compare(gpu, ref, TOL["bf16"], phase)
    xd, dyd = to_device(x, "bf16"), to_device(dy, "bf16")
    names = [n for n in WEIGHTS if n in ref["grads"]]
    # the same gradients once more on top: twice the result
    layer.backward(xd, dyd, phase, accumulate=True)
    torch.cuda.synchronize()
    for n in names:
        check("d" + n, to_host(layer.grads[n]), 2 * ref["grads"][n], TOL["bf16"])
    layer.wgrad_bf16 = True
    for n in WEIGHTS:
        layer.grads[n] = torch.empty_like(layer.grads[n], dtype=torch.bfloat16)
    for times in (1, 2):                                    # stored, then added to
        layer.backward(xd, dyd, phase, accumulate=times == 2)
        torch.cuda.synchronize()
        for n in names:
            check("d" + n, to_host(layer.grads[n]), times * ref["grads"][n], TOL["bf16"])


# hidden, ffn, seq, batch: the products are [T, ffn, hidden], [T, hidden, ffn], [hidden, ffn, T] and their like
SHAPES = [
    (64, 8, 1, 1),            # one token, one chunk of 8
    (128, 72, 65, 1),         # one row past a tile
    (768, 1032, 129, 2),      # 64 x 64 throughout
    (512, 4104, 200, 5),      # 64 x 64, 128 x 128 and 256 x 128, ragged both ways
    (2048, 1544, 1999, 2),    # 256 x 128 and 128 x 128
    (3072, 3848, 2001, 1),    # 256 x 128 and 192 x 256
    (2048, 8200, 2050, 1),    # more large tiles than a round
]


@pytest.mark.parametrize("variant", ["f32 gradients", "bf16 gradients, tanh"])
@pytest.mark.parametrize("hidden,ffn,seq,batch", SHAPES)
def test_bf16_feed_forward_half_on_ragged_sizes(hidden, ffn, seq, batch, variant):
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
def test_bf16_attention_products_on_ragged_sizes(phase, hidden, ffn, seq, batch):
    shape = I.LayerShape(hidden, hidden // 64, ffn, 1, 1, 0, seq, batch, "bf16")
    params = I.full_params(shape, case=520 + batch, random_affine=True)
    x, dy = I.activations(shape, case=520 + batch)
    gpu, ref, _ = run_both(shape, params, x, dy, phase, want_partials=(phase == "both"))
    compare(gpu, ref, TOL["bf16"], phase, want_partials=(phase == "both"))
