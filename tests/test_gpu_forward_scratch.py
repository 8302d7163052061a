"""The forward workspaces that DeviceLayer and DeviceStack keep: one per stream, whatever the layer and micro-batch, with and
without dropout; passes on different streams have different ones."""
import pytest
import torch

from paper_2504_03662_amd import binding as gx
from paper_2504_03662_amd import inputs as I
from paper_2504_03662_amd.runtime import DeviceStack, StageSchedule, cfg_of, one_f_one_b, to_device

pytestmark = pytest.mark.gpu


def _scratch_bytes(stack):
    return sorted(b.numel() for layer in stack.layers for key, b in layer._bufs.items() if "work_fwd" in key)


@pytest.mark.parametrize("drop", [0, 26])
def test_one_workspace_per_stream(drop):
    shape = I.LayerShape(2048, 32, 8192, 1, 1, 0, 64, 1, "bf16", drop_attn=drop, drop_hidden=drop, drop_seed=3 if drop else 0)
    params = [I.full_params(shape, case=860 + k) for k in range(2)]
    need = gx.layer_workspace_bytes(cfg_of(shape), False)
    assert need > 0
    stack = DeviceStack(shape, params)
    xs = [to_device(I.activations(shape, case=870 + m)[0], "bf16") for m in range(3)]
    ys = [stack.forward(x, mb=m).clone() for m, x in enumerate(xs)]
    assert _scratch_bytes(stack) == [need]
    # forward passes that overlap on two streams
    other = torch.cuda.Stream()
    torch.cuda.synchronize()
    for _ in range(3):
        with torch.cuda.stream(other):
            b = stack.forward(xs[1], mb=1)
        a = stack.forward(xs[0], mb=0)
        torch.cuda.synchronize()
        assert torch.equal(a, ys[0]) and torch.equal(b, ys[1])
    assert _scratch_bytes(stack) == [need, need]


def test_stage_with_recomputation_ahead():
    shape = I.LayerShape(512, 8, 1096, 1, 1, 0, 150, 1, "bf16", drop_attn=26, drop_hidden=26, drop_seed=3)
    params = [I.full_params(shape, case=880 + k) for k in range(3)]
    data = [I.activations(shape, case=890 + m) for m in range(3)]
    xs, dys = ([to_device(d[k], "bf16") for d in data] for k in range(2))
    got = []
    for overlap in (False, True):
        stack = DeviceStack(shape, params)
        dxs = []
        StageSchedule(stack, 3, overlap).run(one_f_one_b(3, 2), xs, dys, True, after_backward=lambda m, dx: dxs.append(dx.clone()))
        torch.cuda.synchronize()
        got.append(dxs + [g for layer in stack.layers for g in layer.grads.values()])
        assert len(_scratch_bytes(stack)) == (2 if overlap else 1)
    assert all(torch.equal(a, b) for a, b in zip(*got))


@pytest.mark.parametrize("hidden,ffn,parts", [(2048, 8192, False), (4096, 16384, True)])
def test_a_stage_takes_parts_from_256_mib_of_weights(hidden, ffn, parts):
    shape = I.LayerShape(hidden, hidden // 128, ffn, 1, 1, 0, 64, 1, "bf16")
    assert gx.layer_workspace_bytes(cfg_of(shape), False) > 0                    # a pass on its own takes them
    p = I.full_params(shape, case=861)
    data = [I.activations(shape, case=870 + m) for m in range(2)]
    xs, dys = ([to_device(d[k], "bf16") for d in data] for k in range(2))
    got = []
    for overlap in (False, True):
        for recompute in (False, True):
            stack = DeviceStack(shape, [p])
            dxs = []
            StageSchedule(stack, 2, overlap).run(one_f_one_b(2, 1), xs, dys, recompute,
                                                 after_backward=lambda m, dx: dxs.append(dx.clone()))
            torch.cuda.synchronize()
            got.append(dxs + list(stack.layers[0].grads.values()))
            assert bool(_scratch_bytes(stack)) == parts
    for other in got[1:]:
        assert all(torch.equal(a, b) for a, b in zip(got[0], other))
