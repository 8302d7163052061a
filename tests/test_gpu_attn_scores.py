"""Attention with scores that are set key by key: LayerNorm inputs of +1 and -1 (their normalised values are
the same, exactly) and projections with few entries, so that a chosen component of every key is what a test
asks for and the rounding of q, k and v to bf16 takes no part."""
import numpy as np
import pytest
import torch

from oracle import layer as O
from paper_2504_03662_amd import inputs as I
from paper_2504_03662_amd.runtime import DeviceLayer, to_device, to_host
from parity import TOL, check

pytestmark = pytest.mark.gpu


def _signs(shape, features, seed):
    """Tokens of +1 / -1 with zero mean: `features` [S, n] come first, the rest is random, the second half
    is the negated first."""
    rng = np.random.default_rng(seed)
    half = rng.choice(np.array([-1.0, 1.0], np.float32), (shape.micro_batch, shape.seq, shape.hidden // 2))
    half[:, :, :features.shape[1]] = features
    return np.concatenate([half, -half], axis=2).reshape(shape.tokens, shape.hidden)


def _zero_params(shape):
    p = {n: np.zeros_like(v) for n, v in I.full_params(shape).items()}
    p["ln1_g"][:] = 1.0
    p["ln2_g"][:] = 1.0
    return p


@pytest.mark.parametrize("dh,batch", [(64, 25), (128, 25)])
def test_the_largest_probability_of_a_row_is_not_rounded(dh, batch):
    # 16 heads of 25 samples of one 128-row block: the kernel for many (sample, head) pairs.  Each head
    # gives nearly all weight to key 70 and the rest to key 0, whose score is 1 to 7 powers of 2 lower.
    # Probabilities are taken relative to the largest one, which is then exactly 1; relative to key 0
    # (the maximum of the first 64 keys) it would be a power of 2 with a fractional exponent, whose bf16
    # rounding scales the whole row of the result.  The fitted scale of a row also takes the independent
    # roundings of its 64 or 128 elements, 1.1e-3 / sqrt(64) = 1.4e-4 on the root mean square, and the
    # rounding of the smaller probability times its share.  Worked out on the host with these
    # roundings, the mean over all heads is 1.8e-4, and 8.3e-4 (head dim 64) or 9.7e-4 relative to key 0.
    heads = 16
    shape = I.LayerShape(heads * dh, heads, 64, 1, 1, 0, 128, batch, "bf16")
    h = shape.hidden
    feat = -np.ones((shape.seq, 2), np.float32)
    feat[70, 0] = 1.0
    feat[0, 1] = 1.0
    x = _signs(shape, feat, 700 + dh)
    p = _zero_params(shape)
    rng = np.random.default_rng(701)
    p["w_o"][:] = np.eye(h, dtype=np.float32)
    p["b_qkv"][:h:dh] = 16.0                                       # q = (16, 0, ..)
    p["w_qkv"][0, h:2 * h:dh] = 8.0 + (4 + np.arange(heads)) / 16.0   # k of keys 70, 0: + and - (4 + head) / 16
    p["w_qkv"][1, h:2 * h:dh] = 8.0
    v = I.bf16_round(rng.standard_normal(h).astype(np.float32))
    p["w_qkv"][rng.integers(2, h // 2, h), 2 * h + np.arange(h)] = v   # one entry a column: v = +- the entry
    layer = DeviceLayer(shape, p)
    got = to_host(layer.forward(to_device(x, "bf16"), "attn")["p_attn"])
    ref = O.layer_fwd(shape, p, x, "attn")["p_attn"]
    rows = lambda a: np.asarray(a, np.float64).reshape(batch, 128, heads, dh)[:, 96:]
    got, ref = rows(got), rows(ref)
    scale = (got * ref).sum(-1) / (ref * ref).sum(-1)
    err = float(np.abs(scale - 1).mean())
    print(f"mean error of a row's scale {err:.2e}")
    assert err <= 4e-4
    check("p_attn", got.reshape(-1, h), ref.reshape(-1, h), TOL["bf16"])


@pytest.mark.parametrize("drop", [0, 26])
@pytest.mark.parametrize("dh,heads,batch", [(64, 8, 17), (128, 4, 34), (64, 8, 2), (128, 4, 1)])
def test_scores_that_rise_along_the_keys(dh, heads, batch, drop):
    # Many pairs and few pairs, both head dimensions.  Component 0 of a key is its position / 4, of a query
    # one of two values at random: a row's scores rise by 2 or 3, or by 18 or 26, powers of 2 every 64 keys,
    # both kinds in every wavefront; the other components are ordinary.  Component 0 of dQ and dK is left
    # out, and dx with it: sums of dS times positions up to 63 that cancel, whose error is that of dS in bf16
    # times 63 and not a share of the result.
    shape = I.LayerShape(heads * dh, heads, 64, 1, 1, 0, 300, batch, "bf16", drop_attn=drop,
                         drop_seed=0x5EED if drop else 0)
    h, nbits = shape.hidden, 7
    pos = np.arange(shape.seq) // 4
    rng = np.random.default_rng(710 + dh)
    feat = np.concatenate([2.0 * ((pos[:, None] >> np.arange(nbits)) & 1) - 1, rng.choice([-1.0, 1.0], (shape.seq, 1))],
                          axis=1).astype(np.float32)
    x = _signs(shape, feat, 711)
    p = I.full_params(shape, case=711, random_affine=True)
    p["ln1_g"][:], p["ln1_b"][:] = 1.0, 0.0
    p["w_qkv"][:, :2 * h] = I.bf16_round(p["w_qkv"][:, :2 * h] * np.float32(50 / np.sqrt(h)))
    p["w_qkv"][:, 0:2 * h:dh] = 0.0
    p["b_qkv"][0:2 * h:dh] = 0.0
    for b in range(nbits):
        p["w_qkv"][b, h:2 * h:dh] = 2.0 ** b / 2                   # k component 0: position / 4 - 63.5
    p["w_qkv"][nbits, 0:h:dh] = 4.0
    p["b_qkv"][0:h:dh] = 5.0                                       # q component 0: 1 or 9
    dy = I.activations(shape, case=711)[1]
    layer = DeviceLayer(shape, p)
    xd, dyd = to_device(x, "bf16"), to_device(dy, "bf16")
    got = to_host(layer.forward(xd, "attn")["p_attn"])
    layer.backward(xd, dyd, "attn")
    torch.cuda.synchronize()
    ref = O.layer_fwd(shape, p, x, "attn")
    _, rg = O.layer_bwd(shape, p, dy, ref["cache"], "attn")
    check("p_attn", got, ref["p_attn"], TOL["bf16"])
    kept = np.ones(3 * h, np.float32)
    kept[0:2 * h:dh] = 0.0
    for n in ("w_qkv", "b_qkv"):
        check("d" + n, to_host(layer.grads[n]) * kept, rg[n] * kept, TOL["bf16"])
    check("dw_o", to_host(layer.grads["w_o"]), rg["w_o"], TOL["bf16"])


@pytest.mark.parametrize("dtype,dh,heads,batch", [
    ("bf16", 64, 8, 2), ("bf16", 128, 4, 1), ("bf16", 64, 16, 25), ("bf16", 128, 16, 25), ("f32", 32, 4, 2),
    ("f32", 64, 4, 2), ("f32", 128, 2, 2), ("f32", 20, 4, 2),
])
@pytest.mark.parametrize("star", [1, 6, 66, 70, 93])
def test_one_score_far_above_all_others(dtype, dh, heads, batch, star):
    # 300 (natural) above every other: relative to anything but itself its exponential overflows.  Places 1 to 3
    # of 8 keys are held by one half of a wavefront, 5 to 7 by the other.
    shape = I.LayerShape(heads * dh, heads, 64, 1, 1, 0, 128, batch, dtype)
    h = shape.hidden
    feat = np.zeros((shape.seq, 1), np.float32)
    feat[star] = 1.0
    x = _signs(shape, feat, 720)
    p = I.full_params(shape, case=721, random_affine=True)
    p["ln1_g"][:], p["ln1_b"][:] = 1.0, 0.0
    p["w_qkv"][:, 0:2 * h:dh] = 0.0
    p["b_qkv"][0:2 * h:dh] = 0.0
    p["b_qkv"][0:h:dh] = 16.0                                       # q component 0
    p["w_qkv"][0, h:2 * h:dh] = I.bf16_round(np.float32([300 / 16 * np.sqrt(dh)]))[0]   # k component 0 of the one key
    dy = I.activations(shape, case=722)[1]
    layer = DeviceLayer(shape, p)
    xd, dyd = to_device(x, dtype), to_device(dy, dtype)
    got = to_host(layer.forward(xd, "attn")["p_attn"])
    layer.backward(xd, dyd, "attn")
    torch.cuda.synchronize()
    ref = O.layer_fwd(shape, p, x, "attn")
    _, rg = O.layer_bwd(shape, p, dy, ref["cache"], "attn")
    check("p_attn", got, ref["p_attn"], TOL[dtype])
    kept = np.ones(3 * h, np.float32)                               # as above, without component 0 of dQ and dK
    kept[0:2 * h:dh] = 0.0
    for n in ("w_qkv", "b_qkv"):
        check("d" + n, to_host(layer.grads[n]) * kept, rg[n] * kept, TOL[dtype])
    check("dw_o", to_host(layer.grads["w_o"]), rg["w_o"], TOL[dtype])
