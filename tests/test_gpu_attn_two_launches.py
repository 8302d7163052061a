"""Attention backward passes whose dQ and dK / dV kernels are launched one after the other: values that are not finite in fp32,
repeated bits in bf16, at the lengths of few tiles (with fewer blocks these run in one launch)."""
import numpy as np
import pytest
import torch

from oracle import layer as O
from paper_2504_03662_amd import binding as gx
from paper_2504_03662_amd import inputs as I
from paper_2504_03662_amd.runtime import DeviceLayer, to_device, to_host
from parity import TOL, check, compare, run_both
from test_backward_route_rules import ATTN_ONE_LAUNCH, route

pytestmark = pytest.mark.gpu

HEADS_OF_TWO = [40, 64, 128, 256]             # head dim 20, 32, 64, 128


def _layer(hidden, seq, batch, at, case):
    """a feature that is exactly 0 in every token but number `at` of the last sample; component 0 of every query and key is 0"""
    shape = I.LayerShape(hidden, 2, 8, 1, 1, 0, seq, batch, "f32")
    assert not route(shape, "attn") & ATTN_ONE_LAUNCH
    tokens, dh = shape.tokens, hidden // 2
    half = np.random.default_rng(case).choice(np.array([-1.0, 1.0], np.float32), (tokens, hidden // 2))
    half[:, 0] = 0.0
    half[tokens - seq + at, 0] = 4.0
    p = I.full_params(shape, case=case, random_affine=True)
    p["ln1_g"][:], p["ln1_b"][:] = 1.0, 0.0
    p["w_qkv"][[0, hidden // 2]] = 0.0
    p["w_qkv"][:, 0:2 * hidden:dh] = 0.0
    p["b_qkv"][0:2 * hidden:dh] = 0.0
    return shape, p, np.concatenate([half, -half], axis=1), I.activations(shape, case=case)[1], tokens - seq + at


def _run(shape, p, x, dy):
    layer = DeviceLayer(shape, p)
    xd = to_device(x, "f32")
    layer.forward(xd, "attn")
    dx = to_host(layer.backward(xd, to_device(dy, "f32"), "attn"))
    return dx, {n: to_host(layer.grads[n]) for n in ("w_qkv", "b_qkv")}


@pytest.mark.parametrize("hidden", HEADS_OF_TWO)
def test_fp32_infinite_upstream_gradient_in_a_partial_last_tile(hidden):
    # of the last query of every sample: dV of every key is infinite, and the rows that pad the tile add nothing to it
    shape = I.LayerShape(hidden, 2, 8, 1, 1, 0, 40, 34, "f32")
    assert not route(shape, "attn") & ATTN_ONE_LAUNCH
    p = I.full_params(shape, case=460, random_affine=True)
    x, dy = I.activations(shape, case=460)
    dy[39::40, 3] = np.inf
    got = _run(shape, p, x, dy)[1]["b_qkv"][2 * hidden:]
    np.testing.assert_array_equal(got, np.sign(p["w_o"][:, 3]) * np.float32(np.inf))


@pytest.mark.parametrize("hidden", HEADS_OF_TWO)
@pytest.mark.parametrize("at", [40, 97])                                               # 97: in a partial tile
@pytest.mark.parametrize("what", ["query", "upstream gradient"])
def test_fp32_a_query_that_is_not_finite_stays_from_later_keys(hidden, at, what):
    shape, p, x, dy, row = _layer(hidden, 100, 18, at, 471)
    dx0, _ = _run(shape, p, x, dy)
    if what == "query":
        p["w_qkv"][0, 0:hidden:hidden // 2] = 3e38         # beyond the fp32 range at that token
    else:
        dy[row, 3] = np.inf
    dx1, _ = _run(shape, p, x, dy)
    clean = np.ones(shape.tokens, bool)
    clean[shape.tokens - 100:row + 1] = False
    np.testing.assert_allclose(dx1[clean], dx0[clean], rtol=0, atol=1e-5 * np.abs(dx0).max())
    assert not np.isfinite(dx1[~clean]).all(axis=1).any()


@pytest.mark.parametrize("hidden", HEADS_OF_TWO)
@pytest.mark.parametrize("at", [40, 97])
def test_fp32_a_key_that_is_not_finite_stays_from_earlier_queries(hidden, at):
    # component 0 of one key is -inf and every query's is 1: the key has weight 0
    shape, p, x, dy, row = _layer(hidden, 100, 18, at, 472)
    dh = hidden // 2
    p["w_qkv"][0, hidden:2 * hidden:dh] = -3e38
    p["b_qkv"][0:hidden:dh] = 1.0
    dx, g = _run(shape, p, x, dy)
    assert np.isfinite(dx[:row]).all()
    with np.errstate(over="ignore", invalid="ignore"):
        q = p.copy()
        q["w_qkv"] = p["w_qkv"].astype(np.float64)
        q["w_qkv"][0, hidden:2 * hidden:dh] = -1e308       # -inf in 64 bits as well
        ref = O.layer_fwd(shape, q, x, "attn")
        _, rg = O.layer_bwd(shape, q, dy, ref["cache"], "attn")
    kept = np.ones(3 * hidden, bool)
    kept[0:hidden:dh] = False
    for n in ("w_qkv", "b_qkv"):
        check("d" + n, g[n][..., kept], rg[n][..., kept], TOL["f32"])


@pytest.mark.parametrize("drop", [0, 26])
@pytest.mark.parametrize("dh", [64, 128])
@pytest.mark.parametrize("seq", [1, 33, 65, 97, 129, 255])
def test_bf16_query_tile_counts_repeat_their_bits(seq, dh, drop):
    batch = 257 // (2 * -(-seq // 64)) + 1
    shape = I.LayerShape(2 * dh, 2, 64, 1, 1, 0, seq, batch, "bf16", drop_attn=drop, drop_seed=5 if drop else 0)
    assert not route(shape, "attn") & ATTN_ONE_LAUNCH
    params = I.full_params(shape, case=700 + seq, random_affine=True)
    x, dy = I.activations(shape, case=700 + seq)
    gpu, ref, layer = run_both(shape, params, x, dy, "attn")
    compare(gpu, ref, TOL["bf16"], "attn")
    xd, dyd = to_device(x, "bf16"), to_device(dy, "bf16")
    first = layer.backward(xd, dyd, "attn").clone()
    grad = layer.grads["w_qkv"].clone()
    for _ in range(3):
        assert torch.equal(layer.backward(xd, dyd, "attn"), first)
        assert torch.equal(layer.grads["w_qkv"], grad)
