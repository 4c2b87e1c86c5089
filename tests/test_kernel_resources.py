"""What the compiler gave the kernels of the built library: registers and scratch, from the code objects' own metadata."""
import struct

import pytest

import paper_2605_05049_amd as moe

msgpack = pytest.importorskip("msgpack")
_MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(blob):
    at = blob.find(_MAGIC)
    while at >= 0:
        pos = at + len(_MAGIC)
        (count,) = struct.unpack_from("<Q", blob, pos)
        pos += 8
        for _ in range(count):
            offset, size, length = struct.unpack_from("<3Q", blob, pos)
            triple = blob[pos + 24:pos + 24 + length]
            pos += 24 + length
            if b"gfx950" in triple and size:
                yield blob[at + offset:at + offset + size]
        at = blob.find(_MAGIC, at + 1)


def _kernels(elf):
    """amdhsa.kernels of the AMDGPU metadata note (type 32) of a 64-bit little-endian ELF."""
    (ph_off,) = struct.unpack_from("<Q", elf, 32)
    ph_size, ph_count = struct.unpack_from("<2H", elf, 54)
    for i in range(ph_count):
        kind, _, start, _, _, size = struct.unpack_from("<IIQQQQ", elf, ph_off + i * ph_size)
        pos, end = start, start + size
        while kind == 4 and pos < end:   # PT_NOTE
            n_name, n_desc, note = struct.unpack_from("<3I", elf, pos)
            desc = pos + 12 + (n_name + 3) // 4 * 4
            if note == 32:
                return msgpack.unpackb(elf[desc:desc + n_desc])["amdhsa.kernels"]
            pos = desc + (n_desc + 3) // 4 * 4
    return []


@pytest.fixture(scope="module")
def kernels():
    moe.load_library()
    with open(moe.library_path(), "rb") as f:
        blob = f.read()
    found = {k[".name"]: k for elf in _code_objects(blob) for k in _kernels(elf)}
    assert len(found) > 20
    return found


def test_no_kernel_uses_scratch(kernels):
    """A register that is spilt is a memory round trip in the inner loop: no kernel has one."""
    spilt = {n: (k[".private_segment_fixed_size"], k[".vgpr_spill_count"]) for n, k in kernels.items()
             if k[".private_segment_fixed_size"] or k[".vgpr_spill_count"]}
    assert not spilt


