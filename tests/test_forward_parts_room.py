"""Forward products of few tokens are cut into parts only in a workspace that is known to have the room: sizes without
GX_FWD_PARTS do not shrink when the tokens grow, and the binding sets the flag by the size of the tensor it is given."""
import ctypes
import os

import pytest
import torch

from paper_2504_03662_amd import binding as gx


@pytest.fixture(scope="module", autouse=True)
def lib():
    if not os.path.exists(gx.LIB_PATH):
        from paper_2504_03662_amd.build import build
        build(verbose=False)
    return gx.lib()


def cfg(tokens, drop=0, more=0, hidden=5120, tp=2, batch=1):
    return gx.make_cfg(hidden=hidden, heads=hidden // 128, ffn=4 * hidden, tp_attn=tp, tp_ffn=tp, seq=tokens, micro_batch=batch,
                       dtype=gx.GX_BF16, flags=3 | more | (gx.GX_DROPOUT if drop else 0), drop_attn=drop, drop_hidden=drop)


def c_bytes(c, backward):
    return gx.lib().gx_layer_workspace_bytes(ctypes.byref(c), backward)


@pytest.mark.parametrize("backward,more", [(0, 0), (1, 0), (1, gx.GX_RECOMPUTE)])
@pytest.mark.parametrize("drop", [0, 26])
@pytest.mark.parametrize("hidden,tp", [(5120, 2), (2048, 1), (4096, 8)])
def test_a_block_sized_by_the_longest_sequence_serves_shorter_ones(hidden, tp, drop, backward, more):
    sizes = [c_bytes(cfg(t, drop, more, hidden, tp), backward) for t in range(1, 700)]
    assert sizes == sorted(sizes)
    if not backward and not drop:
        assert not any(sizes)


@pytest.mark.parametrize("drop", [0, 26])
def test_the_flag_follows_the_room_of_the_tensor(drop):
    c = cfg(256, drop)
    need = gx.layer_workspace_bytes(c, False)
    room = lambda n: gx._parts_if_room(c, torch.empty(n, dtype=torch.uint8), False).flags & gx.GX_FWD_PARTS
    assert need >= 30 << 20 and room(need) and not room(need - 1)
    longest = cfg(512, drop)
    assert not room(max(256, gx.layer_workspace_bytes(longest, False)))          # sized by a longer sequence
    assert not c.flags & gx.GX_FWD_PARTS                                         # the caller's own stays as it is
    for unknown in (None, 4096, torch.empty((need, 2), dtype=torch.uint8)[:, 0]):
        assert not gx._parts_if_room(c, unknown, False).flags & gx.GX_FWD_PARTS


@pytest.mark.parametrize("tokens", [1, 32, 64, 128, 256, 257])
def test_a_recomputing_backward_pass_has_room_for_the_parts_beside_the_activations(tokens):
    c = cfg(tokens, 0, gx.GX_RECOMPUTE | gx.GX_FWD_PARTS)
    saved, parts = gx.layer_saved_bytes(c), c_bytes(cfg(tokens, 0, gx.GX_FWD_PARTS), 0)
    assert c_bytes(c, 1) == max(c_bytes(cfg(tokens), 1), parts) + saved
