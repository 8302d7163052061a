"""Which backward passes stay on one stream, launch products in pairs or both attention kernels together (host code)."""
import ctypes
import os

import pytest

from paper_2504_03662_amd import binding as gx
from paper_2504_03662_amd.inputs import LayerShape
from paper_2504_03662_amd.runtime import cfg_of

PAIRS, ONE_STREAM, ATTN_ONE_LAUNCH, FC1_SUMS, QKV_SUMS = 1, 2, 4, 8, 16


@pytest.fixture(scope="module", autouse=True)
def lib():
    if not os.path.exists(gx.LIB_PATH):
        from paper_2504_03662_amd.build import build
        build(verbose=False)
    return gx.lib()


def route(shape, phase="both"):
    return int(gx.lib().gx_bwd_route(ctypes.byref(cfg_of(shape, phase))))


def bf16(hidden, heads, ffn, seq, batch=1, tp=1):
    return LayerShape(hidden, heads, ffn, tp, 1, 0, seq, batch, "bf16")


@pytest.mark.parametrize("phase,shape,one", [
    ("both", bf16(512, 8, 2048, 1024), True), ("both", bf16(512, 8, 2048, 1040), False),             # 3.2 G, and beyond one launch
    ("both", bf16(256, 4, 1024, 256, 7), True), ("both", bf16(256, 4, 1024, 1024, 2), False),        # 1792 tokens, 2048
    ("both", bf16(256, 4, 1024, 1536), False), ("both", bf16(768, 12, 3072, 512), False),
    ("attn", bf16(256, 4, 8, 512, 8), True), ("attn", bf16(256, 4, 8, 512, 9), False),
    ("attn", bf16(768, 6, 8, 8192, 1, 6), False), ("attn", bf16(512, 8, 8, 512, 12, 2), False), ("attn", bf16(256, 4, 8, 2048, 4), False),
    ("mlp", bf16(512, 8, 512, 1024, 6), True), ("mlp", bf16(512, 8, 512, 1025, 6), False),
])
def test_bf16_passes_that_stay_on_one_stream(phase, shape, one):
    want = (ONE_STREAM | (ATTN_ONE_LAUNCH if phase != "mlp" else 0)) if one else 0
    assert route(shape, phase) == want


def test_attention_halves_of_long_sequences_with_two_launches():
    assert route(bf16(256, 4, 8, 2048), "attn") == route(bf16(512, 8, 8, 512, 5), "attn") == ONE_STREAM
    assert route(bf16(256, 4, 8, 2561), "attn") == 0


@pytest.mark.parametrize("hidden,heads,ffn,seq,batch,want", [
    (256, 4, 1024, 128, 2, PAIRS | ATTN_ONE_LAUNCH), (512, 8, 2048, 256, 1, PAIRS | ATTN_ONE_LAUNCH), (512, 8, 2048, 257, 1, ATTN_ONE_LAUNCH),
    (1024, 16, 4096, 512, 2, 0), (128, 4, 256, 64, 32, PAIRS),
])
def test_fp32_passes(hidden, heads, ffn, seq, batch, want):
    assert route(LayerShape(hidden, heads, ffn, 1, 1, 0, seq, batch, "f32")) & 7 == want


@pytest.mark.parametrize("phase,hidden,ffn,seq,want", [
    ("both", 256, 1024, 256, FC1_SUMS | QKV_SUMS), ("both", 1280, 5120, 4096, FC1_SUMS | QKV_SUMS), ("both", 1284, 5136, 608, QKV_SUMS),
    ("both", 2048, 8192, 1024, 0), ("mlp", 256, 1024, 256, FC1_SUMS), ("mlp", 512, 2048, 1024, 0), ("attn", 2048, 64, 256, QKV_SUMS),
    ("attn", 2048, 64, 512, 0),
])
def test_fp32_bias_gradients_in_the_product(phase, hidden, ffn, seq, want):
    assert route(LayerShape(hidden, {1284: 12}.get(hidden, hidden // 64), ffn, 1, 1, 0, seq, 1, "f32"), phase) & 24 == want


@pytest.mark.parametrize("hidden,ffn", [(64, 256), (256, 1024), (324, 1300), (1284, 5136), (2048, 8192)])
def test_fp32_workspace_grows_with_tokens_and_phases(hidden, ffn):
    def size(seq, phase):
        c = cfg_of(LayerShape(hidden, {1284: 12, 324: 3}.get(hidden, hidden // 64), ffn, 1, 1, 0, seq, 1, "f32"), phase)
        return gx.layer_workspace_bytes(c, True)

    sizes = {p: [size(t, p) for t in range(1, 2200, 3)] for p in ("both", "attn", "mlp")}
    assert all(s == sorted(s) for s in sizes.values())
    assert all(b >= max(a, m) for b, a, m in zip(*(sizes[p] for p in ("both", "attn", "mlp"))))


def test_fp32_layers_in_pairs_hold_no_partial_sums_of_bias_gradients():
    T, H, F, blocks = 256, 256, 1024, 16
    c = cfg_of(LayerShape(H, 4, F, 1, 1, 0, T, 1, "f32"))
    assert gx.layer_workspace_bytes(c, True) - 4 * (T * F + 7 * T * H) < 4 * blocks * (F + 5 * H)      # less than they would take
