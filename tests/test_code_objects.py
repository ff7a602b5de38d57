"""What the built library's kernels ask of the GPU, read from the metadata of
its gfx950 code objects: needs no GPU."""
import os
import struct

import msgpack
import pytest

from paper_2503_12450_amd import binding as B

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"
NT_AMDGPU_METADATA, SHT_NOTE = 32, 7


def _code_objects(blob):
    """The gfx950 ELF images of every offload bundle in the library."""
    at = blob.find(MAGIC)
    while at >= 0:
        (n,) = struct.unpack_from("<Q", blob, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(n):
            off, size, name_len = struct.unpack_from("<QQQ", blob, p)
            name = blob[p + 24:p + 24 + name_len]
            p += 24 + name_len
            if b"gfx950" in name:
                yield blob[at + off:at + off + size]
        at = blob.find(MAGIC, at + 1)


def _kernels(elf):
    assert elf[:4] == b"\x7fELF"
    (shoff,) = struct.unpack_from("<Q", elf, 0x28)
    shentsize, shnum = struct.unpack_from("<HH", elf, 0x3A)
    for k in range(shnum):
        _, kind, _, _, off, size = struct.unpack_from("<IIQQQQ", elf, shoff + k * shentsize)
        end = off + size
        while kind == SHT_NOTE and off < end:
            name_len, desc_len, note = struct.unpack_from("<III", elf, off)
            desc = off + 12 + (name_len + 3) // 4 * 4
            if note == NT_AMDGPU_METADATA:
                yield from msgpack.unpackb(elf[desc:desc + desc_len])["amdhsa.kernels"]
            off = desc + (desc_len + 3) // 4 * 4


@pytest.fixture(scope="module")
def kernels():
    with open(B.LIB_PATH, "rb") as f:
        blob = f.read()
    found = [k for elf in _code_objects(blob) for k in _kernels(elf)]
    assert any("attn" in k[".name"] for k in found) and any("gemm" in k[".name"] for k in found)
    return found


def test_no_kernel_needs_scratch_memory(kernels):
    """A kernel that spills registers has a private segment, for which the
    runtime may allocate device memory at its first launch: not under graph
    capture, and not where a call promises to allocate nothing."""
    spilling = {k[".name"]: k[".private_segment_fixed_size"] for k in kernels if k[".private_segment_fixed_size"]}
    assert spilling == {}
