"""Attention with few (sample, head) pairs, whose keys are spread over two wavefronts or, for long sequences, four:
lengths on either side of the rule's 768 keys and of a step's 128, for which a wavefront has no visible key at all,
one step, or an odd or even number of them."""
import pytest
import torch

from paper_2504_03662_amd import inputs as I
from paper_2504_03662_amd.runtime import to_device
from parity import TOL, compare, run_both

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("drop", [0, 26])
@pytest.mark.parametrize("dh,heads", [(64, 2), (128, 1)])
@pytest.mark.parametrize("seq", [767, 768, 769, 833, 991, 1120])
def test_key_shares_against_the_oracle(seq, dh, heads, drop):
    shape = I.LayerShape(heads * dh, heads, 64, 1, 1, 0, seq, 1, "bf16", drop_attn=drop, drop_seed=5 if drop else 0)
    params = I.full_params(shape, case=500 + seq, random_affine=True)
    x, dy = I.activations(shape, case=500 + seq)
    gpu, ref, layer = run_both(shape, params, x, dy, "attn")
    compare(gpu, ref, TOL["bf16"], "attn")
    # and the same bits again, with another call's data in LDS before it
    xd = to_device(x, "bf16")
    first = layer.forward(xd, "attn")["p_attn"].clone()
    for _ in range(3):
        layer.forward(to_device(dy, "bf16"), "attn")
        assert torch.equal(layer.forward(xd, "attn")["p_attn"], first)
