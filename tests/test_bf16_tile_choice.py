"""The tile that a bf16 product takes (host code of the launcher): measured choices, and the sizes that the GPU
tests use to reach every product kernel."""
import os

import pytest

from bf16_tiles import ALL, SHAPES, TILES, reached, tile
from paper_2504_03662_amd import binding as gx


@pytest.fixture(scope="module", autouse=True)
def lib():
    if not os.path.exists(gx.LIB_PATH):
        from paper_2504_03662_amd.build import build
        build(verbose=False)
    return gx.lib()


@pytest.mark.parametrize("m,n,k,expected", [
    (4096, 3072, 4096, "256x192"), (2048, 5120, 10240, "192x256"), (3003, 4096, 2048, "192x256"),
    (2048, 2560, 5120, "256x128"), (4096, 1024, 4096, "128x128"), (512, 4096, 8192, "64x128"),
    (1024, 1024, 4096, "64x64"), (128, 7680, 5120, "64x64"), (2048, 10240, 5120, "256x256 + 128x128"),
    (8192, 8192, 4096, "256x256"), (6618, 1216, 16952, "192x256"),
])
def test_tile_of_measured_products(m, n, k, expected):
    assert tile(m, n, k) == expected


def test_column_sums_stay_with_whole_blocks_of_64_rows():
    for m in range(1, 6000, 187):
        for n in range(8, 9000, 392):
            for k in (64, 1000, 4096):
                assert tile(m, n, k, column_sums=True) not in ("256x192", "192x256")


def test_shapes_of_the_gpu_test_reach_every_product_kernel():
    got = set().union(*[reached(shape, phase) for phase, shape in SHAPES])
    assert got == ALL and len(ALL) == 6 * len(TILES) - 2
