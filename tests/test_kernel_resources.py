"""Registers and spills of the kernels in the built library, from the metadata that the compiler leaves in its code objects."""
import re
import struct

import msgpack
import pytest

from paper_2302_08005_amd import binding as B


def _code_objects(blob):
    """The gfx950 code objects of a library: one bundle per source file."""
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = blob.find(magic)
    while at >= 0:
        (count,), pos = struct.unpack_from("<Q", blob, at + 24), at + 32
        for _ in range(count):
            offset, size, length = struct.unpack_from("<QQQ", blob, pos)
            if b"gfx950" in blob[pos + 24:pos + 24 + length]:
                yield blob[at + offset:at + offset + size]
            pos += 24 + length
        at = blob.find(magic, at + 24)


def _sections(elf):
    """(type, offset, size) of each."""
    shoff, = struct.unpack_from("<Q", elf, 40)
    shentsize, shnum = struct.unpack_from("<HH", elf, 58)
    for i in range(shnum):
        kind, = struct.unpack_from("<I", elf, shoff + i * shentsize + 4)
        yield kind, *struct.unpack_from("<QQ", elf, shoff + i * shentsize + 24)


def _notes(elf):
    for kind, offset, size in _sections(elf):
        if kind == 7:   # SHT_NOTE
            namesz, descsz, note = struct.unpack_from("<III", elf, offset)
            if note == 32:   # NT_AMDGPU_METADATA
                start = offset + 12 + (namesz + 3) // 4 * 4
                yield msgpack.unpackb(elf[start:start + descsz])


@pytest.fixture(scope="module")
def kernels():
    B.lib()
    with open(B.LIB_PATH, "rb") as f:
        found = {k[".name"]: k for elf in _code_objects(f.read()) for meta in _notes(elf) for k in meta["amdhsa.kernels"]}
    assert len(found) > 300
    return found


def _named(kernels, pattern):
    found = {n: k for n, k in kernels.items() if re.search(pattern, n)}
    assert found, pattern
    return found


# a SIMD has 512 registers: two wavefronts where a kernel takes at most 256
@pytest.mark.parametrize("draws", [0, 1])
def test_dq_of_128_wide_heads_runs_two_wavefronts_per_simd(kernels, draws):
    found = _named(kernels, rf"attn_bwd_dq_bf16_kernelILi128ELb{draws}E")
    for half in (0, 1):
        fit = [n for n, k in found.items() if f"ILi128ELb{draws}ELb{half}E" in n and k[".vgpr_count"] <= 256 and k[".vgpr_spill_count"] == 0]
        assert fit, {n: k[".vgpr_count"] for n, k in found.items()}


# dQ and dK/dV with mask draws in one launch, 64-wide heads: all 256 registers of two wavefronts per SIMD, and as few more as can be
@pytest.mark.parametrize("groups,most", [(1, 2), (2, 13)])
def test_spills_of_the_one_launch_backward(kernels, groups, most):
    for name, k in _named(kernels, rf"attn_bwd_both_kernelILi64ELb1ELb[01]ELi{groups}E").items():
        assert k[".vgpr_count"] <= 256 and k[".vgpr_spill_count"] <= most, (name, k[".vgpr_spill_count"])


def test_kernels_start_on_pages():
    """Addresses of the functions in every code object (a step fetches each kernel's code anew, page by page)."""
    with open(B.LIB_PATH, "rb") as f:
        objects = list(_code_objects(f.read()))
    seen = 0
    for elf in objects:
        for kind, offset, size in _sections(elf):
            if kind == 11:   # SHT_DYNSYM
                for at in range(offset, offset + size, 24):
                    info, value = elf[at + 4], struct.unpack_from("<Q", elf, at + 8)[0]
                    if info & 15 == 2:   # STT_FUNC
                        seen += 1
                        assert value % 4096 == 0, hex(value)
    assert seen > 300
