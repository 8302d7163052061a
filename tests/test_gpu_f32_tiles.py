"""fp32 products and attention at the edges of their tiles: remainders of the 32 / 64 row tiles and of
the reduction stages, head dimensions that are padded, every tile size of the dispatch, and values
that are not finite in positions that the causal mask hides."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import layer as O
from paper_2504_03662_amd import binding as gx
from paper_2504_03662_amd import inputs as I
from paper_2504_03662_amd.runtime import DeviceLayer, to_device, to_host
from parity import TOL, check, compare, run_both

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hidden,heads,ffn,seq,batch", [
    (4, 1, 4, 1, 1),            # one token, one chunk
    (36, 3, 20, 31, 1),         # head dim 12, one tile short of a row
    (120, 6, 132, 33, 3),       # head dim 20, one row past a tile
    (100, 2, 200, 65, 2),       # head dim 50: rows that are not multiples of 16 bytes
    (96, 1, 324, 129, 2),       # head dim 96, five key tiles: one wavefront takes two
    (256, 2, 516, 160, 2),      # head dim 128
    (768, 12, 772, 700, 1),     # 64-row tiles, two wavefronts per block
    (512, 8, 2052, 1030, 2),    # 64-row tiles, more than three per compute unit too (one wavefront per block), 33 key tiles
])
def test_fp32_tile_edges(hidden, heads, ffn, seq, batch):
    shape = I.LayerShape(hidden, heads, ffn, 1, 1, 0, seq, batch, "f32")
    params = I.full_params(shape, case=400 + seq, random_affine=True)
    x, dy = I.activations(shape, case=400 + seq)
    gpu, ref, _ = run_both(shape, params, x, dy, want_partials=True)
    compare(gpu, ref, TOL["f32"], want_partials=True)


def _tile(m, n, k):
    f = gx.lib().gx_f32_tile
    f.argtypes, f.restype = [ctypes.c_int] * 3, ctypes.c_int
    return f(m, n, k)


def test_fp32_one_wavefront_per_block_ragged_reductions():
    # 64-row tiles with one wavefront per block in all three layouts, each with an odd number of stages of 32 reduction
    # steps whose last one is not whole, and a weight gradient of four stages; stored and added to
    shape = I.LayerShape(1036, 14, 4100, 1, 1, 0, 1030, 1, "f32")
    t, h, f = shape.tokens, shape.hidden, shape.ffn
    assert {_tile(t, 3 * h, h), _tile(t, f, h), _tile(h, f, t)} == {2}      # NN; NN and NT; TN
    assert all(-(-k // 32) % 2 == 1 and k % 32 for k in (h, t))
    params = I.full_params(shape, case=480, random_affine=True)
    x, dy = I.activations(shape, case=480)
    gpu, ref, layer = run_both(shape, params, x, dy, want_partials=True)
    compare(gpu, ref, TOL["f32"], want_partials=True)
    layer.backward(to_device(x, "f32"), to_device(dy, "f32"), accumulate=True)
    torch.cuda.synchronize()
    for n in I.PARAM_NAMES:
        np.testing.assert_array_equal(to_host(layer.grads[n]), 2 * gpu["grads"][n])


@pytest.mark.parametrize("tokens", [1, 31, 64, 97, 160, 161])
def test_fp32_weight_gradients_of_few_tokens(tokens):
    # the kernels for short reductions, one to five stages of 32 or 64 steps, whole and not, and one token beyond
    shape = I.LayerShape(516, 6, 2060, 1, 1, 0, tokens, 1, "f32")
    long = tokens > 160
    assert _tile(516, 1548, tokens) == (1 if long else 3) and _tile(516, 2060, tokens) == (1 if long else 4)
    params = I.full_params(shape, case=490 + tokens, random_affine=True)
    x, dy = I.activations(shape, case=490 + tokens)
    gpu, ref, layer = run_both(shape, params, x, dy, want_partials=True)
    compare(gpu, ref, TOL["f32"], want_partials=True)
    layer.backward(to_device(x, "f32"), to_device(dy, "f32"), accumulate=True)
    torch.cuda.synchronize()
    for n in I.PARAM_NAMES:
        np.testing.assert_array_equal(to_host(layer.grads[n]), 2 * gpu["grads"][n])


def test_fp32_accumulation_and_dropout_with_padded_heads():
    shape = I.LayerShape(144, 3, 164, 1, 1, 0, 77, 2, "f32", drop_attn=40, drop_hidden=30, drop_seed=0xABCDEF0123)
    params = I.full_params(shape, case=431, random_affine=True)
    x, dy = I.activations(shape, case=431)
    gpu, ref, layer = run_both(shape, params, x, dy, want_partials=True)
    compare(gpu, ref, TOL["f32"], want_partials=True)
    xd, dyd = to_device(x, "f32"), to_device(dy, "f32")
    layer.backward(xd, dyd, accumulate=True)
    torch.cuda.synchronize()
    for n in I.PARAM_NAMES:
        # twice one backward pass: each element is one fp32 addition of equal values, exact
        np.testing.assert_array_equal(to_host(layer.grads[n]), 2 * gpu["grads"][n])


@pytest.mark.parametrize("heads", [1, 2, 4, 8])
@pytest.mark.parametrize("at", [40, 99])
def test_fp32_values_that_are_not_finite_stay_behind_the_mask(heads, at):
    # one token of one sample is not finite: rows before it are untouched (up to the order of their sums),
    # the other sample bit for bit, its own row is not finite
    shape = I.LayerShape(256, heads, 256, 1, 1, 0, 100, 2, "f32") if heads > 1 else \
        I.LayerShape(128, heads, 256, 1, 1, 0, 100, 2, "f32")
    params = I.full_params(shape, case=440, random_affine=True)
    x, dy = I.activations(shape, case=440)
    layer = DeviceLayer(shape, params)
    dyd = to_device(dy, "f32")
    xd = to_device(x, "f32")
    y0 = to_host(layer.forward(xd)["y"])
    xbad = x.copy()
    xbad[at] = np.inf
    xb = to_device(xbad, "f32")
    y1 = to_host(layer.forward(xb)["y"])
    dx1 = to_host(layer.backward(xb, dyd))
    layer.forward(xd)
    dx0 = to_host(layer.backward(xd, dyd))
    # the tile that holds the token adds its finite rows in another order, so equal up to rounding there
    tol = dict(rtol=0, atol=1e-5 * np.abs(y0).max())
    np.testing.assert_allclose(y1[:at], y0[:at], **tol)
    np.testing.assert_array_equal(y1[100:], y0[100:])
    np.testing.assert_array_equal(dx1[100:], dx0[100:])
    assert not np.isfinite(y1[at]).any()


def _with_keys_out_of_range(hidden, heads, seq, keys):
    """A layer whose scores are -inf in fp32 for the keys named, and ordinary for all others: component 0
    of every query is 1e20, of those keys -1e20, of the others exactly 0 (a feature that is 0 there in tokens
    of +1 and -1 with zero mean, which LayerNorm leaves 0)."""
    shape = I.LayerShape(hidden, heads, 8, 1, 1, 0, seq, 2, "f32")
    rng = np.random.default_rng(450)
    half = rng.choice(np.array([-1.0, 1.0], np.float32), (shape.micro_batch, seq, hidden // 2))
    half[:, :, 0] = np.isin(np.arange(seq), keys)
    x = np.concatenate([half, -half], axis=2).reshape(shape.tokens, hidden)
    p = I.full_params(shape, case=450, random_affine=True)
    dh = hidden // heads
    p["ln1_g"][:], p["ln1_b"][:] = 1.0, 0.0
    p["w_qkv"][[0, hidden // 2]] = 0.0
    p["w_qkv"][:, 0:2 * hidden:dh] = 0.0
    p["w_qkv"][0, hidden:2 * hidden:dh] = -1e20
    p["b_qkv"][0:hidden:dh] = 1e20
    p["b_qkv"][hidden:2 * hidden:dh] = 0.0
    return shape, p, x


@pytest.mark.parametrize("hidden,heads", [(40, 2), (64, 2), (128, 2), (256, 2)])       # head dim 20, 32, 64, 128
@pytest.mark.parametrize("keys", [[32], range(32, 64), [64, 65, 95, 129], range(0, 32), range(0, 64)])
def test_fp32_keys_whose_scores_are_minus_infinity_get_no_weight(hidden, heads, keys):
    # also where they are all that a wavefront sees of its first tile, or of every tile; a query that sees
    # no other key has no result
    keys = list(keys)
    shape, p, x = _with_keys_out_of_range(hidden, heads, 160, keys)
    first = 0 if keys[0] > 0 else keys[-1] + 1
    dy = I.activations(shape, case=451)[1]
    layer = DeviceLayer(shape, p)
    xd, dyd = to_device(x, "f32"), to_device(dy, "f32")
    got = to_host(layer.forward(xd, "attn")["p_attn"]).reshape(2, 160, hidden)
    with np.errstate(over="ignore", invalid="ignore"):
        ref = O.layer_fwd(shape, p, x, "attn")
    check("p_attn", got[:, first:].reshape(-1, hidden), ref["p_attn"].reshape(2, 160, hidden)[:, first:].reshape(-1, hidden),
          TOL["f32"])
    if first:
        assert not np.isfinite(got[:, :first]).any()
        return
    layer.backward(xd, dyd, "attn")
    torch.cuda.synchronize()
    with np.errstate(over="ignore", invalid="ignore"):
        _, g = O.layer_bwd(shape, p, dy, ref["cache"], "attn")
    kept = np.ones(3 * hidden, bool)               # without component 0 of Q and K, which holds the 1e20s
    kept[0:2 * hidden:hidden // heads] = False
    for n in ("w_qkv", "b_qkv"):
        check("d" + n, to_host(layer.grads[n])[..., kept], g[n][..., kept], TOL["f32"])
    check("dw_o", to_host(layer.grads["w_o"]), g["w_o"], TOL["f32"])


@pytest.mark.parametrize("hidden,heads", [(40, 2), (64, 2), (128, 2), (256, 2)])       # head dim 20, 32, 64, 128
def test_fp32_infinite_upstream_gradient_in_a_partial_last_tile(hidden, heads):
    # the last query's upstream gradient is infinite in one column, its gradient of the heads' outputs then
    # in all of them, and so is dV = P^T dO of every key, with the sign that dO has: the rows that pad the
    # last tile add nothing to it
    shape = I.LayerShape(hidden, heads, 8, 1, 1, 0, 40, 1, "f32")
    p = I.full_params(shape, case=460, random_affine=True)
    x, dy = I.activations(shape, case=460)
    dy[-1, 3] = np.inf
    layer = DeviceLayer(shape, p)
    xd = to_device(x, "f32")
    layer.forward(xd, "attn")
    layer.backward(xd, to_device(dy, "f32"), "attn")
    got = to_host(layer.grads["b_qkv"])[2 * hidden:]
    np.testing.assert_array_equal(got, np.sign(p["w_o"][:, 3]) * np.float32(np.inf))


def _one_token_layer(hidden, heads, at):
    """A layer with a feature that is exactly 0 in every token but `at` (tokens of +1 and -1 with zero mean)."""
    shape = I.LayerShape(hidden, heads, 8, 1, 1, 0, 100, 1, "f32")
    half = np.random.default_rng(470).choice(np.array([-1.0, 1.0], np.float32), (100, hidden // 2))
    half[:, 0] = 0.0
    half[at, 0] = 4.0
    p = I.full_params(shape, case=470, random_affine=True)
    dh = hidden // heads
    p["ln1_g"][:], p["ln1_b"][:] = 1.0, 0.0
    p["w_qkv"][[0, hidden // 2]] = 0.0
    p["w_qkv"][:, 0:2 * hidden:dh] = 0.0               # component 0 of every query and key: 0
    p["b_qkv"][0:2 * hidden:dh] = 0.0
    return shape, p, np.concatenate([half, -half], axis=1)


def _run_attn(shape, p, x, dy):
    layer = DeviceLayer(shape, p)
    xd = to_device(x, "f32")
    layer.forward(xd, "attn")
    dx = to_host(layer.backward(xd, to_device(dy, "f32"), "attn"))
    return dx, {n: to_host(layer.grads[n]) for n in ("w_qkv", "b_qkv")}


@pytest.mark.parametrize("hidden,heads", [(40, 2), (64, 2), (128, 2), (256, 2)])       # head dim 20, 32, 64, 128
@pytest.mark.parametrize("at", [40, 97])                                               # 97: in a partial tile
@pytest.mark.parametrize("what", ["query", "upstream gradient"])
def test_fp32_a_query_that_is_not_finite_stays_from_later_keys(hidden, heads, at, what):
    # dK and dV of the keys after it, which it does not see, and with them dx of those tokens
    shape, p, x = _one_token_layer(hidden, heads, at)
    dy = I.activations(shape, case=470)[1]
    dx0, _ = _run_attn(shape, p, x, dy)
    if what == "query":
        p["w_qkv"][0, 0:hidden:hidden // heads] = 3e38     # beyond the fp32 range at that token
    else:
        dy[at, 3] = np.inf
    dx1, _ = _run_attn(shape, p, x, dy)
    np.testing.assert_allclose(dx1[at + 1:], dx0[at + 1:], rtol=0, atol=1e-5 * np.abs(dx0).max())
    assert not np.isfinite(dx1[:at + 1]).all(axis=1).any()


@pytest.mark.parametrize("hidden,heads", [(40, 2), (64, 2), (128, 2), (256, 2)])
@pytest.mark.parametrize("at", [40, 97])
def test_fp32_a_key_that_is_not_finite_stays_from_earlier_queries(hidden, heads, at):
    # component 0 of one key is -inf and every query's is 1: the key has weight 0, and only dQ of the queries
    # that see it is not finite, in that component
    shape, p, x = _one_token_layer(hidden, heads, at)
    dh = hidden // heads
    p["w_qkv"][0, hidden:2 * hidden:dh] = -3e38
    p["b_qkv"][0:hidden:dh] = 1.0
    dy = I.activations(shape, case=470)[1]
    dx, g = _run_attn(shape, p, x, dy)
    assert np.isfinite(dx[:at]).all()
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
