"""fp32 attention, backward: dQ and dK / dV in one launch (D formed by both) and in two, on either side of the lines between them,
with padded head dimensions, a partial last tile and dropout."""
import pytest

from paper_2504_03662_amd import inputs as I
from parity import TOL, compare, run_both

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("drop", [0, 40])
@pytest.mark.parametrize("heads,dh,seq,batch", [
    (1, 4, 1, 1), (2, 20, 33, 3), (4, 50, 65, 2), (2, 100, 129, 2),
    (4, 64, 1024, 1),           # 128 blocks of 32 rows
    (17, 64, 225, 1),           # 136 of 17 pairs: two launches
    (8, 32, 1030, 2),           # 528 of 16 pairs, head dim 32: two launches
    (8, 32, 1024, 2),           # 512
    (2, 128, 700, 1),
])
def test_fp32_attention_backward(heads, dh, seq, batch, drop):
    more = dict(drop_attn=drop, drop_seed=0x9876543210) if drop else {}
    shape = I.LayerShape(heads * dh, heads, 8, 1, 1, 0, seq, batch, "f32", **more)
    params = I.full_params(shape, case=630 + seq, random_affine=True)
    x, dy = I.activations(shape, case=630 + seq)
    gpu, ref, _ = run_both(shape, params, x, dy, "attn")
    compare(gpu, ref, TOL["f32"], "attn")
