"""The dK / dV kernel works on three query tiles of 32 at once: lengths for which a pair of wavefronts has no tile, one,
two, three, or an odd or even number of them, with a last tile of one row, of all but one, or whole; more than one sample,
so that a tile beyond a sample's end may not read the next one's rows; repeated, the same bits.  The short ones run in one
launch with dQ; on their own: test_gpu_attn_two_launches.py."""
import pytest
import torch

from paper_2504_03662_amd import inputs as I
from paper_2504_03662_amd.runtime import to_device
from parity import TOL, compare, run_both
from test_attn_key_shares_rule import key_shares

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("drop", [0, 26])
@pytest.mark.parametrize("dh", [64, 128])
@pytest.mark.parametrize("seq", [1, 31, 32, 33, 64, 65, 95, 96, 97, 128, 129, 161, 255])
def test_query_tile_counts_against_the_oracle(seq, dh, drop):
    shape = I.LayerShape(2 * dh, 2, 64, 1, 1, 0, seq, 2, "bf16", drop_attn=drop, drop_seed=5 if drop else 0)
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


@pytest.mark.parametrize("drop", [0, 26])
@pytest.mark.parametrize("dh", [64, 128])
@pytest.mark.parametrize("seq", [2047, 2048, 2113])
def test_dq_key_shares_of_one_pair_against_the_oracle(seq, dh, drop):
    # from 2048 keys on the dQ kernel spreads few pairs' keys over four wavefronts instead of two
    shape = I.LayerShape(dh, 1, 64, 1, 1, 0, seq, 1, "bf16", drop_attn=drop, drop_seed=5 if drop else 0)
    params = I.full_params(shape, case=900 + seq, random_affine=True)
    x, dy = I.activations(shape, case=900 + seq)
    gpu, ref, layer = run_both(shape, params, x, dy, "attn")
    compare(gpu, ref, TOL["bf16"], "attn")


@pytest.mark.parametrize("drop", [0, 26])
@pytest.mark.parametrize("dh,heads,batch,seq", [(64, 2, 3, 2049), (128, 2, 2, 2113), (128, 6, 1, 2800), (64, 3, 2, 2950)])
def test_four_key_shares_of_several_heads_and_samples(dh, heads, batch, seq, drop):
    # both kernels with four shares: pair -> (head, sample), steps of 128 keys that end beyond a sample's last row, and (the
    # last two) more than 256 workgroups; again on other data's LDS, the same bits
    assert key_shares(batch, seq, heads, dh, False) == key_shares(batch, seq, heads, dh, True) == 4
    shape = I.LayerShape(dh * heads, heads, 64, 1, 1, 0, seq, batch, "bf16", drop_attn=drop, drop_seed=5 if drop else 0)
    params = I.full_params(shape, case=950 + seq, random_affine=True)
    x, dy = I.activations(shape, case=950 + seq)
    gpu, ref, layer = run_both(shape, params, x, dy, "attn")
    compare(gpu, ref, TOL["bf16"], "attn")
    xd, dyd = to_device(x, "bf16"), to_device(dy, "bf16")
    out = layer.forward(xd, "attn")["p_attn"].clone()
    first = layer.backward(xd, dyd, "attn").clone()
    grad = layer.grads["w_qkv"].clone()
    for _ in range(3):
        layer.forward(dyd, "attn")
        assert torch.equal(layer.forward(xd, "attn")["p_attn"], out)
        assert torch.equal(layer.backward(xd, dyd, "attn"), first)
        assert torch.equal(layer.grads["w_qkv"], grad)
