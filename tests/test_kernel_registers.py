"""Registers of the attention kernels, read from the metadata of the built library: no bf16 kernel spills, and the ones of
256 threads at head dim 64 leave room for three wavefronts per SIMD (512 / 3 registers, in steps of 8), but for the one that
holds both backward kernels, which is for layers of at most two workgroups per compute unit; fp32 kernels spill where the
source says so, and no more."""
import os
import struct

import msgpack
import pytest

from paper_2504_03662_amd import binding as gx
from test_static_scratch_symbol import _code_objects


def _metadata(elf):
    """the amdhsa.kernels list of an ELF64 code object (note 32 of owner AMDGPU, a msgpack map)"""
    phoff, = struct.unpack_from("<Q", elf, 0x20)
    phentsize, phnum = struct.unpack_from("<HH", elf, 0x36)
    for i in range(phnum):
        ptype, _, off, _, _, size = struct.unpack_from("<IIQQQQ", elf, phoff + i * phentsize)
        pos = off
        while ptype == 4 and pos < off + size:                 # PT_NOTE
            nlen, dlen, kind = struct.unpack_from("<III", elf, pos)
            data = pos + 12 + (nlen + 3) // 4 * 4
            if kind == 32 and elf[pos + 12:pos + 12 + nlen].rstrip(b"\0") == b"AMDGPU":
                return msgpack.unpackb(elf[data:data + dlen], raw=False)["amdhsa.kernels"]
            pos = data + (dlen + 3) // 4 * 4
    return []


@pytest.fixture(scope="module")
def kernels():
    if not os.path.exists(gx.LIB_PATH):
        from paper_2504_03662_amd.build import build
        build(verbose=False)
    found = {}
    for triple, elf in _code_objects(open(gx.LIB_PATH, "rb").read()):
        if "gfx950" in triple and elf[:4] == b"\x7fELF":
            found.update({k[".name"]: k for k in _metadata(elf)})
    return found


def _of(kernels, dh, name):
    got = {n: k for n, k in kernels.items() if f"4dh{dh}" in n.replace("5dh128", "4dh128") and name in n}
    assert got
    return got


@pytest.mark.parametrize("dh", [64, 128])
@pytest.mark.parametrize("name", ["attn_bwd_dq_kernel", "attn_bwd_dkv_kernel", "attn_fwd_kernel", "attn_bwd_both_kernel"])
def test_attention_kernels_do_not_spill(kernels, dh, name):
    for n, k in _of(kernels, dh, name).items():
        assert k[".vgpr_spill_count"] == 0 and k[".private_segment_fixed_size"] == 0, n


@pytest.mark.parametrize("name", ["attn_bwd_dq_kernel", "attn_bwd_dkv_kernel", "attn_fwd_kernel"])
def test_three_wavefronts_per_simd_at_head_dim_64(kernels, name):
    for n, k in _of(kernels, 64, name).items():
        if k[".max_flat_workgroup_size"] == 256:
            assert k[".vgpr_count"] <= 168, n


# registers spilled, by the kernel's padded head dimension and whether the head dimension fills it
F32_SPILLS = {("attn_bwd_dkv_f32_kernel", 128, True): 43, ("attn_bwd_dkv_f32_kernel", 128, False): 28,
              ("attn_bwd_f32_kernel", 128, True): 94, ("attn_bwd_f32_kernel", 128, False): 34,
              ("attn_bwd_dq_f32_kernel", 64, False): 1}


@pytest.mark.parametrize("name", ["attn_fwd_f32_kernel", "attn_bwd_dq_f32_kernel", "attn_bwd_dkv_f32_kernel", "attn_bwd_f32_kernel"])
@pytest.mark.parametrize("dh", [32, 64, 128])
@pytest.mark.parametrize("exact", [True, False])
def test_fp32_attention_kernels_spill_no_more_than_stated(kernels, name, dh, exact):
    got = [k for n, k in kernels.items() if f"{len(name)}{name}ILi{dh}ELb{int(exact)}E" in n]
    assert len(got) == 1
    assert got[0][".vgpr_spill_count"] <= F32_SPILLS.get((name, dh, exact), 0)
