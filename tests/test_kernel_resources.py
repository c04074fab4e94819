"""Registers and scratch memory of the built kernels, from the metadata of the library's code objects."""
import re
import struct

import msgpack
import pytest

from paper_2603_30033_amd import binding as ta

# kernels whose working set does not fit 256 registers a lane
SPILLS = [
    "attn_prefill_kernelIfLi128E", "bwd_dq_kernelIfLi128E",      # 128 channels in fp32
    "attn_merge_kernelILi2ELi[234]E",                            # merged latents of 64 to 128 channels beside two heads of 64
]


def code_objects(blob):
    """The gfx950 ELF images of every offload bundle in the library."""
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = blob.find(magic)
    while at >= 0:
        p = at + len(magic)
        count, = struct.unpack_from("<Q", blob, p)
        p += 8
        for _ in range(count):
            offset, size, length = struct.unpack_from("<QQQ", blob, p)
            if b"gfx950" in blob[p + 24:p + 24 + length] and size:
                yield blob[at + offset:at + offset + size]
            p += 24 + length
        at = blob.find(magic, at + 1)


def kernels(elf):
    """Metadata of every kernel: the AMDGPU note (type 32) of the image's note sections (type 7)."""
    sections, = struct.unpack_from("<Q", elf, 40)
    entry, count = struct.unpack_from("<HH", elf, 58)
    for i in range(count):
        kind, = struct.unpack_from("<I", elf, sections + i * entry + 4)
        at, size = struct.unpack_from("<QQ", elf, sections + i * entry + 24)
        end = at + size
        while kind == 7 and at < end:
            name, desc, note = struct.unpack_from("<III", elf, at)
            start = at + 12 + (name + 3) // 4 * 4
            if note == 32 and elf[at + 12:at + 12 + name].rstrip(b"\0") == b"AMDGPU":
                yield from msgpack.unpackb(elf[start:start + desc])["amdhsa.kernels"]
            at = start + (desc + 3) // 4 * 4


@pytest.fixture(scope="module")
def built():
    ta.load_library()
    blob = open(ta.LIB_PATH, "rb").read()
    return [k for elf in code_objects(blob) for k in kernels(elf)]


def test_only_the_widest_kernels_use_scratch_memory(built):
    names = [k[".name"] for k in built]
    for part in ("decode_proj_kernel", "decode_qhat_kernel", "decode_attn_kernel", "attn_prefill_kernel", "gemm_kernel", "bwd_dkv_kernel"):
        assert any(part in n for n in names), part
    for pattern in SPILLS:
        assert any(re.search(pattern, n) for n in names), pattern
    for k in built:
        if not any(re.search(pattern, k[".name"]) for pattern in SPILLS):
            assert k[".private_segment_fixed_size"] == 0 and k[".vgpr_spill_count"] == 0, k[".name"]
