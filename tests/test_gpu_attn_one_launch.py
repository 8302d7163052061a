"""bf16 attention, backward, on either side of the line between one launch for dQ and dK / dV (up to 1024 keys, up to 256
blocks of 64 keys, small layers) and two; the lengths of few query tiles also with more blocks than that."""
import pytest

from paper_2504_03662_amd import inputs as I
from parity import TOL, compare, run_both

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("drop", [0, 26])
@pytest.mark.parametrize("dh", [64, 128])
@pytest.mark.parametrize("heads,seq,batch", [
    (2, 1024, 1), (1, 1025, 2),                               # the longest, and one more
    (2, 1000, 8), (17, 961, 1),                               # 256 blocks, and 272
    (2, 1, 130), (2, 33, 130), (2, 64, 130), (1, 65, 131), (1, 97, 130), (1, 129, 87),     # beyond 256 blocks, few tiles
])
def test_attention_backward_launches(dh, heads, seq, batch, drop):
    shape = I.LayerShape(heads * dh, heads, 64, 1, 1, 0, seq, batch, "bf16", drop_attn=drop, drop_seed=7 if drop else 0)
    params = I.full_params(shape, case=720 + seq, random_affine=True)
    x, dy = I.activations(shape, case=720 + seq)
    gpu, ref, _ = run_both(shape, params, x, dy, "attn")
    compare(gpu, ref, TOL["bf16"], "attn")
