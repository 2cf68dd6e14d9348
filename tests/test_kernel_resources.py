"""CPU: what the built kernels ask of the register file.  A workgroup of the main kernels fills its share of it, and a
value that the compiler moves to scratch memory is read back inside the key loop, where the read waits for every
staging load in flight: no kernel of the library may have one."""
import struct
from pathlib import Path

import msgpack
import pytest

pv = pytest.importorskip("paper_2605_04263_amd.binding")

BUNDLE = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(blob):
    """The gfx950 ELF images in a host library."""
    at = blob.find(BUNDLE)
    while at >= 0:
        entry = at + len(BUNDLE) + 8
        for _ in range(struct.unpack_from("<Q", blob, at + len(BUNDLE))[0]):
            offset, size, name_len = struct.unpack_from("<QQQ", blob, entry)
            if size and b"gfx950" in blob[entry + 24:entry + 24 + name_len]:
                yield blob[at + offset:at + offset + size]
            entry += 24 + name_len
        at = blob.find(BUNDLE, at + 1)


def kernels(elf):
    """The metadata entries of an image: the note sections hold them as MessagePack."""
    section = struct.unpack_from("<Q", elf, 0x28)[0]
    size, count = struct.unpack_from("<HH", elf, 0x3A)
    for i in range(count):
        header = section + i * size
        if struct.unpack_from("<I", elf, header + 4)[0] == 7:                 # SHT_NOTE
            note = struct.unpack_from("<Q", elf, header + 0x18)[0]
            name, length, _ = struct.unpack_from("<III", elf, note)
            start = note + 12 + (name + 3) // 4 * 4
            yield from msgpack.unpackb(elf[start:start + length])["amdhsa.kernels"]


def test_no_kernel_uses_scratch_memory():
    found = [k for elf in code_objects(Path(pv.LIB_PATH).read_bytes()) for k in kernels(elf)]
    # both head sizes: eight group sizes and the query-tile workgroups, with and without the rotation
    assert sum("k_attn_bf16" in k[".name"] for k in found) == 2 * 9 * 2
    assert any("k_attn_fp8" in k[".name"] for k in found)
    bad = {k[".name"]: (k[".private_segment_fixed_size"], k[".vgpr_spill_count"]) for k in found
           if k[".private_segment_fixed_size"] or k[".vgpr_spill_count"]}
    assert not bad, bad
