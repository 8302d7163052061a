"""Which attention kernel (sample, head) pairs and lengths take, host code of the launcher: measured choices, on either side of
each line."""
import ctypes
import os

import pytest

from paper_2504_03662_amd import binding as gx


@pytest.fixture(scope="module", autouse=True)
def lib():
    if not os.path.exists(gx.LIB_PATH):
        from paper_2504_03662_amd.build import build
        build(verbose=False)
    return gx.lib()


def key_shares(batch, seq, heads, dh, backward):
    f = gx.lib().gx_attn_key_shares
    f.argtypes, f.restype = [ctypes.c_int] * 5, ctypes.c_int
    return f(batch, seq, heads, dh, int(backward))


@pytest.mark.parametrize("pairs,seq,expected", [
    (12, 767, 2), (12, 768, 4), (16, 1024, 4), (16, 1025, 2), (16, 2048, 2), (15, 1089, 4), (12, 2048, 4), (8, 4096, 4),
    (4, 8192, 4), (5, 8192, 2), (48, 1024, 2), (49, 1024, 1), (64, 2048, 1)])
@pytest.mark.parametrize("dh", [64, 128])
def test_forward(pairs, seq, expected, dh):
    assert key_shares(pairs, seq, 1, dh, False) == expected
    assert key_shares(1, seq, pairs, dh, False) == expected


@pytest.mark.parametrize("pairs,seq,dh128,dh64", [
    (2, 2047, 2, 2), (2, 2048, 4, 4), (8, 2048, 4, 4), (9, 2048, 2, 2), (7, 4096, 4, 4), (8, 4096, 2, 2), (4, 8192, 4, 4),
    (5, 8192, 2, 4), (6, 8192, 2, 4), (7, 8192, 1, 1), (5, 6528, 4, 4), (5, 6592, 2, 4), (48, 1024, 2, 2), (49, 1024, 1, 1)])
def test_dq(pairs, seq, dh128, dh64):
    assert key_shares(pairs, seq, 1, 128, True) == key_shares(1, seq, pairs, 128, True) == dh128
    assert key_shares(pairs, seq, 1, 64, True) == key_shares(1, seq, pairs, 64, True) == dh64
