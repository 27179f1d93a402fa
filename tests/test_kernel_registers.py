"""Registers of the kernels as built: none keeps a vector register in scratch memory.  A scratch access is a load that the
matrix-core kernels' counted waits do not count.  And where their LDS begins."""
import os
import re
import struct

import pytest

from paper_2602_10940_amd import binding as B


msgpack = pytest.importorskip("msgpack")


def _code_objects(path):
    """The gfx950 ELF images in the offload bundles of a library."""
    data = open(path, "rb").read()
    at = data.find(b"__CLANG_OFFLOAD_BUNDLE__")
    while at >= 0:
        p = at + 32
        for _ in range(struct.unpack_from("<Q", data, at + 24)[0]):
            off, size, length = struct.unpack_from("<QQQ", data, p)
            if b"gfx950" in data[p + 24:p + 24 + length] and size:
                yield data[at + off:at + off + size]
            p += 24 + length
        at = data.find(b"__CLANG_OFFLOAD_BUNDLE__", at + 24)


def _kernels(elf):
    """The kernel descriptions of the AMDGPU metadata note (type 32, a msgpack map)."""
    shoff, = struct.unpack_from("<Q", elf, 40)
    shentsize, shnum = struct.unpack_from("<HH", elf, 58)
    for i in range(shnum):
        kind, = struct.unpack_from("<I", elf, shoff + i * shentsize + 4)
        p, size = struct.unpack_from("<QQ", elf, shoff + i * shentsize + 24)
        end = p + size
        while kind == 7 and p < end:                       # SHT_NOTE
            name, desc, note = struct.unpack_from("<III", elf, p)
            p += 12 + (name + 3) // 4 * 4
            if note == 32:
                yield from msgpack.unpackb(elf[p:p + desc])["amdhsa.kernels"]
            p += (desc + 3) // 4 * 4


def test_no_kernel_spills_a_vector_register():
    if not os.path.exists(B.LIB_PATH):
        from paper_2602_10940_amd import build
        build.build()
    kernels = [k for elf in _code_objects(B.LIB_PATH) for k in _kernels(elf)]
    assert sum("attn_pp" in k[".name"] for k in kernels) >= 36 and sum("attn_tile" in k[".name"] for k in kernels) >= 30
    spilled = {k[".name"]: (k[".vgpr_spill_count"], k[".private_segment_fixed_size"]) for k in kernels
               if k[".vgpr_spill_count"] or k[".private_segment_fixed_size"]}
    assert not spilled


def test_lds_of_the_matrix_core_kernels_begins_at_a_multiple_of_64():
    """d = 64 finds half of V's rows by XOR of a whole LDS address with 32.  What the compiler puts in front of the array (256 bytes for
    __syncthreads_or today) is not for the source to say, so the array has to ask for it."""
    text = open(os.path.join(os.path.dirname(B.LIB_PATH), "csrc", "attn_mfma.hip")).read()
    asked = re.findall(r"extern __shared__ __align__\((\w+)\)", text)
    values = [int(x) if x.isdigit() else int(re.search(r"constexpr int %s = (\d+);" % x, text).group(1)) for x in asked]
    assert len(values) == text.count("extern __shared__") == 2 and all(v % 64 == 0 for v in values)
