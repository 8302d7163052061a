"""bf16 forward passes of few tokens, whose products' reductions are cut into parts: the edges of the three tiles, ragged widths
and reductions, the halves alone, dropout, guard bytes behind the workspace, and the same call without a workspace."""
import pytest
import torch

from paper_2504_03662_amd import binding as gx
from paper_2504_03662_amd import inputs as I
from paper_2504_03662_amd.runtime import DeviceLayer, cfg_of, to_device, to_host
from oracle import layer as O
from parity import TOL, check

pytestmark = pytest.mark.gpu


def _forward(layer, x, phase, guard=4096):
    cfg = cfg_of(layer.shape, phase)
    n = gx.layer_workspace_bytes(cfg, False)
    ws = torch.full((n + guard,), 0x5A, dtype=torch.uint8, device="cuda:0")
    saved = torch.empty(gx.layer_saved_bytes(cfg), dtype=torch.uint8, device="cuda:0")
    out = {k: layer.empty_act() for k in {"both": ("y", "p_attn", "p_mlp"), "attn": ("p_attn",), "mlp": ("p_mlp",)}[phase]}
    args = [out.get(k) for k in ("y", "p_attn", "p_mlp")]
    gx.layer_fwd(cfg, layer.params, x, *args, saved, ws, torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert n > 0 and bool((ws[n:] == 0x5A).all())
    return {k: to_host(v) for k, v in out.items()}, cfg, saved


@pytest.mark.parametrize("phase,hidden,ffn,seq,batch,drop", [
    ("both", 2048, 8192, 1, 1, 0), ("both", 2048, 8200, 63, 1, 0), ("both", 2112, 6000, 32, 2, 26), ("both", 1984, 10248, 65, 1, 0),
    ("both", 2048, 8192, 64, 2, 26), ("attn", 3584, 8, 127, 1, 0), ("mlp", 1088, 23000, 97, 1, 0), ("mlp", 4096, 16400, 129, 1, 0),
    ("mlp", 4096, 16400, 128, 2, 0), ("both", 4096, 8328, 65, 1, 0), ("both", 4096, 8328, 256, 1, 0),   # plain: reads ahead
])
def test_split_products_against_the_oracle(phase, hidden, ffn, seq, batch, drop):
    shape = I.LayerShape(hidden, hidden // 64, ffn, 1, 1, 0, seq, batch, "bf16", drop_attn=drop, drop_hidden=drop,
                         drop_seed=11 if drop else 0)
    params = I.full_params(shape, case=810 + seq, random_affine=True)
    x, _ = I.activations(shape, case=810 + seq)
    layer = DeviceLayer(shape, params)
    xd = to_device(x, "bf16")
    got, cfg, saved = _forward(layer, xd, phase)
    ref = O.layer_fwd(shape, params, x, phase, True, True)
    for k, v in got.items():
        check(k, v, ref[k], TOL["bf16"])
    again, _, saved2 = _forward(layer, xd, phase)
    for k, v in got.items():
        assert (v == again[k]).all()                        # the parts are added in their order
    if not drop:                                            # one launch per product: another order of additions
        plain = {k: layer.empty_act() for k in got}
        gx.layer_fwd(cfg, layer.params, xd, *[plain.get(k) for k in ("y", "p_attn", "p_mlp")], saved2, None,
                     torch.cuda.current_stream().cuda_stream)
        torch.cuda.synchronize()
        for k, v in plain.items():
            check(k, to_host(v), ref[k], TOL["bf16"])


@pytest.mark.parametrize("drop", [0, 26])
def test_a_workspace_sized_by_a_longer_sequence_is_not_written_past(drop):
    shape = I.LayerShape(2048, 32, 8192, 1, 1, 0, 64, 1, "bf16", drop_attn=drop, drop_hidden=drop, drop_seed=5 if drop else 0)
    params = I.full_params(shape, case=830, random_affine=True)
    x, _ = I.activations(shape, case=830)
    layer = DeviceLayer(shape, params)
    n = max(256, gx.layer_workspace_bytes(cfg_of(shape.with_(seq=200)), False))
    cfg = cfg_of(shape)
    assert n < gx.layer_workspace_bytes(cfg, False)
    block = torch.full((gx.layer_workspace_bytes(cfg, False) + 4096,), 0x5A, dtype=torch.uint8, device="cuda:0")
    saved, y = torch.empty(gx.layer_saved_bytes(cfg), dtype=torch.uint8, device="cuda:0"), layer.empty_act()
    gx.layer_fwd(cfg, layer.params, to_device(x, "bf16"), y, None, None, saved, block[:n], torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert bool((block[n:] == 0x5A).all())
    check("y", to_host(y), O.layer_fwd(shape, params, x, "both", True, True)["y"], TOL["bf16"])
