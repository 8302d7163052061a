"""LayerNorm forward and backward at row lengths on either side of each launch shape (wavefronts per row,
chunks per lane), with row counts that leave workgroups without a full step."""
import pytest

from paper_2504_03662_amd import inputs as I
from parity import TOL, compare, run_both

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,hidden", [
    ("bf16", 64), ("bf16", 512), ("bf16", 576), ("bf16", 1024), ("bf16", 2048), ("bf16", 2112), ("bf16", 4096),
    ("bf16", 4160), ("bf16", 8192), ("f32", 4), ("f32", 256), ("f32", 260), ("f32", 1024), ("f32", 1028), ("f32", 2052),
    ("f32", 4096),
])
@pytest.mark.parametrize("rows", [1, 67])
def test_layer_norm_launch_shapes(dtype, hidden, rows):
    heads = hidden // 64 if hidden % 64 == 0 else hidden // 4
    shape = I.LayerShape(hidden, heads, 64, heads, 1, 0, rows, 1, dtype)     # one local head: a small unused half
    params = I.rank_params(shape, case=600 + rows, random_affine=True)
    x, dy = I.activations(shape, case=600 + rows)
    gpu, ref, _ = run_both(shape, params, x, dy, "mlp")
    compare(gpu, ref, TOL[dtype], "mlp")


@pytest.mark.parametrize("dtype,hidden,rows", [
    ("bf16", 2112, 2048), ("bf16", 2112, 2049), ("bf16", 3072, 4096), ("bf16", 2560, 4097), ("f32", 1028, 2049),
    ("f32", 1536, 2050), ("f32", 1280, 7168), ("f32", 1028, 7169),
])
def test_layer_norm_rows_of_five_and_six_chunks_per_lane(dtype, hidden, rows):
    # one wavefront per row or four, by the number of rows
    test_layer_norm_launch_shapes(dtype, hidden, rows)
