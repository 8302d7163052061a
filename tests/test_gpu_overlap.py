"""Backward passes that hand work to the library's side stream (by the rule's own word: gx_bwd_route): the same bits as on one
stream, from a captured graph, and from two host threads; whole blocks, halves alone, with accumulation and dropout, fp32."""
import threading

import pytest
import torch

from paper_2504_03662_amd import binding as gx
from paper_2504_03662_amd import inputs as I
from paper_2504_03662_amd.runtime import DeviceLayer, to_device
from test_backward_route_rules import ONE_STREAM, PAIRS, route

pytestmark = pytest.mark.gpu

CASES = [("both", "bf16", 0), ("both", "bf16", 26), ("attn", "bf16", 0), ("mlp", "bf16", 0), ("both", "f32", 0), ("mlp", "f32", 0)]


def _layer(phase, dtype, drop, case):
    hidden, heads, ffn, seq = (1024, 8, 4096, 520) if dtype == "bf16" else (516, 6, 2064, 150)
    shape = I.LayerShape(hidden, heads, ffn, 1, 1, 0, seq, 2, dtype, drop_attn=drop, drop_hidden=drop, drop_seed=9 if drop else 0)
    assert not route(shape, phase) & (ONE_STREAM | PAIRS)             # it forks
    x, dy = I.activations(shape, case=case)
    return DeviceLayer(shape, I.full_params(shape, case=case, random_affine=True)), to_device(x, dtype), to_device(dy, dtype)


def _bits(t):
    return t.view(torch.int16) if t.dtype == torch.bfloat16 else t.view(torch.int32)


def _same(a, b):
    return all(torch.equal(_bits(p), _bits(q)) for p, q in zip(a, b))


@pytest.mark.parametrize("accumulate", [False, True])
@pytest.mark.parametrize("phase,dtype,drop", CASES)
def test_side_stream_changes_no_bit(phase, dtype, drop, accumulate):
    layer, x, dy = _layer(phase, dtype, drop, 980)
    layer.forward(x, phase)

    def backward():
        for g in layer.grads.values():
            g.fill_(0.125)
        dx = layer.backward(x, dy, phase, accumulate=accumulate)
        return [dx] + [g.clone() for g in layer.grads.values()]

    with_side = [backward() for _ in range(3)]
    gx.set_overlap(False)
    try:
        serial = backward()
    finally:
        gx.set_overlap(True)
    assert serial[0].float().abs().sum() > 0 and all(_same(serial, w) for w in with_side)


@pytest.mark.parametrize("accumulate", [False, True])
@pytest.mark.parametrize("phase,dtype,drop", CASES)
def test_forks_and_joins_replay_from_a_captured_graph(phase, dtype, drop, accumulate):
    layer, x, dy = _layer(phase, dtype, drop, 981)
    out, dx = layer.empty_act(), layer.empty_act()

    def step():
        layer.forward(x, phase, out=out)
        layer.backward(x, dy, phase, accumulate=accumulate, out=dx)

    def reset():
        for t in (out, dx, *layer.grads.values()):
            t.fill_(0.5)
        torch.cuda.synchronize()

    def snapshot():
        torch.cuda.synchronize()
        return [t.clone() for t in (out, dx, *layer.grads.values())]

    step()                                     # creates the side stream, its events and the buffers
    reset()
    step()
    want = snapshot()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        step()
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    for _ in range(3):
        reset()
        graph.replay()
        assert _same(snapshot(), want)
        reset()
        step()                                 # eager work between replays
        assert _same(snapshot(), want)


@pytest.mark.parametrize("phase", ["both", "mlp"])
def test_two_host_threads_have_their_own_side_streams(phase):
    def run(reps, out):
        layer, x, dy = _layer(phase, "bf16", 0, 982)
        with torch.cuda.stream(torch.cuda.Stream()):
            for _ in range(reps):
                layer.forward(x, phase)
                dx = layer.backward(x, dy, phase)
            torch.cuda.current_stream().synchronize()
        out.append([dx] + list(layer.grads.values()))

    alone, res = [], [[], []]
    run(1, alone)
    torch.cuda.synchronize()
    threads = [threading.Thread(target=run, args=(20, r)) for r in res]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    assert all(_same(r[0], alone[0]) for r in res)
