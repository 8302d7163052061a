"""The tile that an fp32 product takes (host code of the launcher): measured choices on either side of each line."""
import ctypes
import os

import pytest

from paper_2504_03662_amd import binding as gx


@pytest.mark.parametrize("m,n,k,expected", [
    (512, 1024, 1024, 0), (512, 1024, 33, 0), (512, 1032, 1024, 1), (1024, 1024, 160, 3), (1024, 1024, 161, 1),
    (1024, 1028, 33, 4), (1024, 1028, 161, 1), (1536, 2048, 128, 4), (1536, 2048, 8192, 1), (1536, 2052, 192, 2),
    (1536, 2052, 160, 4), (1024, 4096, 1024, 2)])
def test_tile_of_measured_products(m, n, k, expected):
    if not os.path.exists(gx.LIB_PATH):
        from paper_2504_03662_amd.build import build
        build(verbose=False)
    f = gx.lib().gx_f32_tile
    f.argtypes, f.restype = [ctypes.c_int] * 3, ctypes.c_int
    assert f(m, n, k) == expected
