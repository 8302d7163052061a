"""Recomputed activations at sizes whose forward products are cut into parts: gradients with GX_RECOMPUTE, also with the static
workspace, and the saved block of GX_FWD_SAVED_ONLY hold the forward pass's own bits."""
import pytest
import torch

from paper_2504_03662_amd import binding as gx
from paper_2504_03662_amd import inputs as I
from paper_2504_03662_amd.runtime import DeviceLayer, cfg_of, to_device

pytestmark = pytest.mark.gpu


def _bits(t):
    return t.view(torch.int16) if t.dtype == torch.bfloat16 else t


@pytest.mark.parametrize("phase,hidden,ffn,seq,batch,drop", [
    ("both", 2048, 8192, 64, 1, 0), ("both", 2048, 8200, 33, 1, 0), ("both", 2048, 8192, 32, 2, 26), ("both", 4096, 8328, 65, 1, 0),
    ("attn", 3584, 8, 64, 1, 0), ("mlp", 8192, 8200, 200, 1, 0),
])
def test_recomputed_activations_have_the_bits_of_the_forward_pass(phase, hidden, ffn, seq, batch, drop):
    shape = I.LayerShape(hidden, hidden // 64, ffn, 1, 1, 0, seq, batch, "bf16", drop_attn=drop, drop_hidden=drop,
                         drop_seed=11 if drop else 0)
    params = I.full_params(shape, case=840 + seq, random_affine=True)
    x, dy = I.activations(shape, case=840 + seq)
    layer = DeviceLayer(shape, params)
    xd, dyd = to_device(x, "bf16"), to_device(dy, "bf16")
    assert gx.layer_workspace_bytes(cfg_of(shape, phase), False) >= 4 * shape.tokens * hidden * 2     # at least two parts
    for key in ("saved", "only"):                 # bytes between the pieces are nobody's
        layer._buf(key, gx.layer_saved_bytes(cfg_of(shape, phase))).zero_()
    layer.forward(xd, phase)
    layer.forward(xd, phase, saved_key="only", saved_only=True)
    a, b = layer._bufs["saved"], layer._bufs["only"]
    dx = layer.backward(xd, dyd, phase).clone()
    grads = {n: g.clone() for n, g in layer.grads.items()}
    assert torch.isfinite(dx).all() and dx.abs().sum() > 0

    def same(dx2):
        assert torch.equal(_bits(dx2), _bits(dx))
        for n, g in grads.items():
            assert torch.equal(layer.grads[n], g), n

    assert torch.equal(a, b)
    for g in layer.grads.values():
        g.zero_()
    same(layer.backward(xd, dyd, phase, saved_key="only"))
    for g in layer.grads.values():
        g.zero_()
    same(layer.backward(xd, dyd, phase, recompute=True))
    cfg = cfg_of(shape, phase, recompute=True)
    if gx.layer_workspace_bytes(cfg, True) <= 64 << 20:
        for g in layer.grads.values():
            g.zero_()
        out = layer.empty_act()
        gx.layer_bwd_static(cfg, layer.params, xd, dyd, out, layer.grads, None, torch.cuda.current_stream().cuda_stream)
        same(out)
