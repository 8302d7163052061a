"""Forward products of few tokens in calls with many weights have workgroups that only read the next product's weights
(the rule is host code: test_bf16_read_ahead_rule.py): all three products with and without it, last chunks that are not
whole, and calls of other sizes and phases around it, which read nothing ahead; repeated, the same bits.  DeviceLayer gives a
workspace, with which such products are cut into parts instead; reading ahead is for calls without one."""
import pytest
import torch

from oracle import layer as O
from paper_2504_03662_amd import binding as gx
from paper_2504_03662_amd import inputs as I
from paper_2504_03662_amd.runtime import DeviceLayer, cfg_of, to_device, to_host
from parity import TOL, check, compare, run_both
from test_bf16_read_ahead_rule import forward_workgroups

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


@pytest.mark.parametrize("tokens,expected", [(65, (64, 128, 124)), (144, (64, 64, 0)), (256, (64, 0, 124))])
def test_products_that_read_ahead_against_the_oracle(tokens, expected):
    shape = I.LayerShape(4096, 32, 8328, 1, 1, 0, tokens, 1, "bf16")        # weights of 270 MB
    assert forward_workgroups(4096, 4096, 8328, tokens) == expected
    params = I.full_params(shape, case=850 + tokens, random_affine=True)
    x, dy = I.activations(shape, case=850 + tokens)
    gpu, ref, layer = run_both(shape, params, x, dy, "both", recompute=tokens == 144)
    compare(gpu, ref, TOL["bf16"], "both")
    xd = to_device(x, "bf16")
    first = layer.forward(xd, "both")["y"].clone()
    for _ in range(3):
        assert torch.equal(layer.forward(xd, "both")["y"], first)


@pytest.mark.parametrize("tokens,expected", [(65, (64, 128, 124)), (144, (64, 64, 0)), (256, (64, 0, 124))])
def test_calls_without_a_workspace_read_ahead(tokens, expected):
    shape = I.LayerShape(4096, 32, 8328, 1, 1, 0, tokens, 1, "bf16")        # weights of 270 MB
    assert forward_workgroups(4096, 4096, 8328, tokens) == expected
    cfg = cfg_of(shape)
    assert gx.layer_workspace_bytes(cfg, False, parts=False) == 0 < gx.layer_workspace_bytes(cfg, False)
    params = I.full_params(shape, case=850 + tokens, random_affine=True)
    x, _ = I.activations(shape, case=850 + tokens)
    layer = DeviceLayer(shape, params)
    xd, y = to_device(x, "bf16"), layer.empty_act()
    saved = torch.zeros(gx.layer_saved_bytes(cfg), dtype=torch.uint8, device="cuda:0")

    def forward():
        gx.layer_fwd(cfg, layer.params, xd, y, None, None, saved, None, torch.cuda.current_stream().cuda_stream)
        return y.clone(), saved.clone()

    first = forward()
    check("y", to_host(first[0]), O.layer_fwd(shape, params, x, "both", True, True)["y"], TOL["bf16"])
    for _ in range(3):
        again = forward()
        assert torch.equal(again[0], first[0]) and torch.equal(again[1], first[1])
