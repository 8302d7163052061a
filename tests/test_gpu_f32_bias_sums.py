"""fp32 bias gradients of layers whose products are not launched in pairs: added up by the weight gradient, by a pass over the
tensor, and one of each; stored and added to."""
import numpy as np
import pytest
import torch

from paper_2504_03662_amd import inputs as I
from paper_2504_03662_amd.runtime import to_device, to_host
from parity import TOL, compare, run_both
from test_backward_route_rules import FC1_SUMS, PAIRS, QKV_SUMS, route

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("phase,hidden,heads,ffn,seq,sums", [
    ("both", 324, 3, 2052, 290, FC1_SUMS | QKV_SUMS), ("both", 1284, 12, 5136, 608, QKV_SUMS), ("mlp", 324, 3, 2052, 290, 0),
    ("attn", 516, 12, 64, 290, QKV_SUMS), ("attn", 2048, 16, 64, 330, 0),
])
def test_bias_gradients(phase, hidden, heads, ffn, seq, sums):
    shape = I.LayerShape(hidden, heads, ffn, 1, 1, 0, seq, 1, "f32")
    assert route(shape, phase) & (PAIRS | FC1_SUMS | QKV_SUMS) == sums
    params = I.full_params(shape, case=660 + seq, random_affine=True)
    x, dy = I.activations(shape, case=660 + seq)
    gpu, ref, layer = run_both(shape, params, x, dy, phase)
    compare(gpu, ref, TOL["f32"], phase)
    layer.backward(to_device(x, "f32"), to_device(dy, "f32"), phase, accumulate=True)
    torch.cuda.synchronize()
    for n in ref["grads"]:
        np.testing.assert_array_equal(to_host(layer.grads[n]), 2 * gpu["grads"][n])
