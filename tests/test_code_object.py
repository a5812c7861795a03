"""What the compiler made of the kernels, from the metadata in the built library's own gfx950 code objects."""
import os
import struct

import msgpack
import pytest

from paper_2509_25762_amd import binding as ob


def code_objects(data):
    """The device ELF images in the offload bundles of a library."""
    at = data.find(b"__CLANG_OFFLOAD_BUNDLE__")
    while at >= 0:
        count, = struct.unpack_from("<Q", data, at + 24)
        entry = at + 32
        for _ in range(count):
            offset, size, length = struct.unpack_from("<QQQ", data, entry)
            if data[entry + 24:entry + 24 + length].startswith(b"hip") and size:
                yield data[at + offset:at + offset + size]
            entry += 24 + length
        at = data.find(b"__CLANG_OFFLOAD_BUNDLE__", at + 24)


def kernels_of(elf):
    """The kernels of an image, as the metadata note lists them."""
    sections, = struct.unpack_from("<Q", elf, 40)
    for i in range(struct.unpack_from("<H", elf, 60)[0]):
        kind, = struct.unpack_from("<I", elf, sections + 64 * i + 4)
        if kind == 7:   # SHT_NOTE
            offset, = struct.unpack_from("<Q", elf, sections + 64 * i + 24)
            name, desc, _ = struct.unpack_from("<III", elf, offset)
            begin = offset + 12 + (name + 3) // 4 * 4
            yield from msgpack.unpackb(elf[begin:begin + desc])["amdhsa.kernels"]


@pytest.fixture(scope="module")
def attention_kernels():
    if not os.path.exists(ob.LIB_PATH):
        from paper_2509_25762_amd import build
        build.build(verbose=False)
    found = {k[".name"]: k for e in code_objects(open(ob.LIB_PATH, "rb").read()) for k in kernels_of(e) if "attn_" in k[".name"]}
    assert sum("attn_fwd_kernel" in n for n in found) >= 16 and len(found) >= 28
    return found


def test_attention_kernels_spill_no_vector_register(attention_kernels):
    for name, k in attention_kernels.items():
        assert k[".vgpr_spill_count"] == 0 and k[".private_segment_fixed_size"] == 0, name


def test_attention_kernels_spill_few_scalars(attention_kernels):
    """A masked unit compares 8 or 16 registers with the columns' limits.  Formed all at once the results do not fit the
    scalar registers: 159 and 161 spills in the append variants with two column blocks, with reads and writes in every
    masked unit.  One at a time, what is left (up to 14) is written in front of the loops and read on their rare paths."""
    for name, k in attention_kernels.items():
        assert k[".sgpr_spill_count"] <= 24, (name, k[".sgpr_spill_count"])
