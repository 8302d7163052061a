"""fp32 layers so small that the backward pass launches each input gradient together with a weight gradient: reductions that
two stages of 128 steps hold and longer ones, remainders of the 32 x 32 tiles, halves on their own, gradients added to, and the
first size that is no longer launched so."""
import numpy as np
import pytest
import torch

from paper_2504_03662_amd import inputs as I
from paper_2504_03662_amd.runtime import to_device, to_host
from parity import TOL, compare, run_both

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("phase", ["both", "attn", "mlp"])
@pytest.mark.parametrize("hidden,heads,ffn,seq", [
    (128, 4, 256, 128),         # whole tiles, one stage
    (132, 3, 256, 129),         # one past a tile and past a stage
    (252, 2, 260, 256),         # two stages and beyond
    (256, 4, 2048, 250),        # the largest feed-forward width
    (256, 4, 2052, 250),        # beyond it
    (64, 1, 36, 1000),          # a reduction of many stages
])
def test_fp32_paired_products(phase, hidden, heads, ffn, seq):
    shape = I.LayerShape(hidden, heads, ffn, 1, 1, 0, seq, 1, "f32")
    params = I.full_params(shape, case=610 + seq, random_affine=True)
    x, dy = I.activations(shape, case=610 + seq)
    gpu, ref, layer = run_both(shape, params, x, dy, phase)
    compare(gpu, ref, TOL["f32"], phase)
    layer.backward(to_device(x, "f32"), to_device(dy, "f32"), phase, accumulate=True)
    torch.cuda.synchronize()
    for n in ref["grads"]:
        np.testing.assert_array_equal(to_host(layer.grads[n]), 2 * gpu["grads"][n])
