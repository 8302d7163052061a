"""Cutting the reduction of a forward product into parts (host code): every part has something to do, all of them find a compute
unit at once, and the scratch is asked for where it pays."""
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


def parts(m, n, k):
    f = gx.lib().gx_bf16_split
    f.argtypes, f.restype = [ctypes.c_int] * 3, ctypes.c_int
    return f(m, n, k)


def test_parts():
    assert parts(128, 10240, 5120) == 3 and parts(128, 5120, 10240) == 6 and parts(128, 7680, 5120) == 4
    assert parts(128, 16392, 5120) == 1 and parts(257, 5120, 10240) == 1 and parts(128, 5120, 256) == 1
    for n in list(range(8, 2000, 56)) + list(range(2000, 17000, 1064)):
        for k in (8, 64, 250, 264, 1000, 2560, 5120, 10248, 28672):
            p = parts(128, n, k)
            assert p >= 1 and -(-n // 128) * p <= max(256, -(-n // 128))
            if p > 1:
                steps = [s for s in range(256, k + 256, 128) if -(-k // s) == p]
                assert steps and (p - 1) * steps[0] < k       # no part is empty


@pytest.mark.parametrize("hidden,heads,ffn,tp,tokens,asked", [
    (5120, 40, 20480, 2, 1, True), (5120, 40, 20480, 2, 256, True), (5120, 40, 20480, 2, 257, False),
    (2048, 16, 8192, 1, 128, True), (2048, 16, 8192, 1, 129, False), (4096, 32, 16384, 8, 64, True),
    (4096, 32, 16384, 8, 65, False), (1024, 16, 4096, 1, 1, False),
])
def test_where_it_pays(hidden, heads, ffn, tp, tokens, asked):
    c = gx.make_cfg(hidden=hidden, heads=heads, ffn=ffn, tp_attn=tp, tp_ffn=tp, tp_rank=0, seq=tokens, micro_batch=1,
                    dtype=gx.GX_BF16, flags=3)
    assert (gx.layer_workspace_bytes(c, False) > 0) == asked
    c.flags |= gx.GX_FWD_SAVED_ONLY
    assert gx.layer_workspace_bytes(c, False) == 0
