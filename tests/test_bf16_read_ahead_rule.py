"""How many workgroups of a forward product read the next product's weights ahead (host code of the launcher): none where
the call's weights may still be in the memory-side cache, where what is read would be gone before its use, where tokens are
too few or too many, or where nearly all compute units have a tile."""
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


def forward_workgroups(hidden, hidden_local, ffn_local, tokens):
    """of the QKV, output and FC1 products of a whole block, each followed by the next one's weights"""
    f = gx.lib().gx_bf16_read_ahead
    f.argtypes, f.restype = [ctypes.c_int] * 3 + [ctypes.c_long] * 2, ctypes.c_int
    call = 2 * (4 * hidden * hidden_local + 2 * hidden * ffn_local)
    fc = 2 * hidden * ffn_local
    return (f(tokens, 3 * hidden_local, hidden, 2 * hidden_local * hidden, call), f(tokens, hidden, hidden_local, fc, call),
            f(tokens, ffn_local, hidden, fc, call))


@pytest.mark.parametrize("hidden,hidden_local,ffn_local", [(2048, 2048, 8192), (4096, 1024, 4096), (8192, 1024, 3584),
                                                            (1024, 1024, 4104), (5120, 1280, 5120), (4096, 4096, 8192)])
def test_nothing_is_read_ahead_where_the_weights_of_the_call_may_be_cached(hidden, hidden_local, ffn_local):
    assert 2 * (4 * hidden * hidden_local + 2 * hidden * ffn_local) <= 256 << 20
    for tokens in range(1, 1100, 7):
        assert forward_workgroups(hidden, hidden_local, ffn_local, tokens) == (0, 0, 0)


@pytest.mark.parametrize("hidden,hidden_local,ffn_local", [(8192, 4096, 14336), (5120, 5120, 20480)])
def test_nothing_is_read_ahead_that_would_be_gone_before_its_use(hidden, hidden_local, ffn_local):
    for tokens in range(1, 1100, 7):
        assert forward_workgroups(hidden, hidden_local, ffn_local, tokens)[1:] == (0, 0)


@pytest.mark.parametrize("tokens,expected", [(1, (0, 0, 0)), (64, (0, 0, 0)), (65, (16, 96, 96)), (128, (16, 96, 96)),
                                             (256, (0, 96, 96)), (257, (0, 0, 0)), (1024, (0, 0, 0))])
def test_tokens(tokens, expected):
    assert forward_workgroups(5120, 2560, 10240, tokens) == expected


def test_beyond_128_tokens_a_quarter_of_the_compute_units_is_idle_wherever_something_is_read():
    for hidden, local, ffn in ((5120, 2560, 10240), (4096, 4096, 16384), (6144, 3072, 12288), (8192, 2048, 7168)):
        for tokens in range(129, 600):
            assert all(n == 0 or 64 <= n < 256 for n in forward_workgroups(hidden, local, ffn, tokens))
