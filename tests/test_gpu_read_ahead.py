"""Forward products of few tokens have workgroups that only read the next product's weights, from 8 MB of them on: a
last chunk that is not whole, either side of the 8 MB and of the 1024 tokens up to which it is done, in each phase;
repeated, the same bits."""
import pytest
import torch

from paper_2504_03662_amd import inputs as I
from paper_2504_03662_amd.runtime import to_device
from parity import TOL, compare, run_both

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("phase,recompute", [("both", False), ("both", True), ("attn", False), ("mlp", False)])
@pytest.mark.parametrize("hidden,ffn,tokens", [(1024, 4088, 64), (1024, 4096, 1), (1024, 4104, 200), (1024, 4104, 1024),
                                                (1024, 4104, 1025), (2048, 2056, 130)])
def test_few_tokens_against_the_oracle(hidden, ffn, tokens, phase, recompute):
    shape = I.LayerShape(hidden, hidden // 64, ffn, 1, 1, 0, tokens, 1, "bf16")
    params = I.full_params(shape, case=800 + tokens, random_affine=True)
    x, dy = I.activations(shape, case=800 + tokens)
    gpu, ref, layer = run_both(shape, params, x, dy, phase, recompute=recompute)
    compare(gpu, ref, TOL["bf16"], phase)
    xd = to_device(x, "bf16")
    out = "y" if phase == "both" else "p_" + phase
    first = layer.forward(xd, phase)[out].clone()
    for _ in range(3):
        assert torch.equal(layer.forward(xd, phase)[out], first)
