"""Registers of the compiled kernels, from the metadata that the compiler leaves in the library.

A vector register kept in scratch inside a main loop costs more than its load: the wait for it counts every request of memory, so
it also waits for the tiles that have just been asked for."""
import struct

import msgpack

from paper_2503_15758_amd import build as lib_build


def _code_objects(data):
    at = data.find(b"__CLANG_OFFLOAD_BUNDLE__")
    while at >= 0:
        (n,), p = struct.unpack_from("<Q", data, at + 24), at + 32
        for _ in range(n):
            off, size, name = struct.unpack_from("<QQQ", data, p)
            if b"gfx950" in data[p + 24:p + 24 + name]:
                yield data[at + off:at + off + size]
            p += 24 + name
        at = data.find(b"__CLANG_OFFLOAD_BUNDLE__", at + 24)


def _kernels(elf):
    (sections,), (width, count) = struct.unpack_from("<Q", elf, 40), struct.unpack_from("<HH", elf, 58)
    for i in range(count):
        kind, _, _, off, size = struct.unpack_from("<IQQQQ", elf, sections + i * width + 4)
        end = off + size
        while kind == 7 and off < end:                          # SHT_NOTE
            name, desc, note = struct.unpack_from("<III", elf, off)
            body = off + 12 + (name + 3) // 4 * 4
            if note == 32:                                      # NT_AMDGPU_METADATA
                yield from msgpack.unpackb(elf[body:body + desc], strict_map_key=False)["amdhsa.kernels"]
            off = body + (desc + 3) // 4 * 4


def test_no_vector_register_is_kept_in_scratch():
    data = open(lib_build.LIB, "rb").read()
    kernels = [k for elf in _code_objects(data) for k in _kernels(elf)]
    assert len(kernels) > 100
    spilled = {k[".name"]: k[".vgpr_spill_count"] for k in kernels if k[".vgpr_spill_count"]}
    assert not spilled, spilled


def test_the_forward_does_not_keep_a_condition_per_masked_score():
    """Each is compared and used at once; kept in pairs of scalar registers, as the compiler does with stores under conditions that
    imply each other, they take 73 to 94 of them where 75 are enough for all, and the masked step of a short walk 1 to 4 % of its time."""
    data = open(lib_build.LIB, "rb").read()
    in_order = [k for elf in _code_objects(data) for k in _kernels(elf) if "fwd_mfma_kernel" in k[".name"] and "ELb0EE" in k[".name"]]
    assert len(in_order) == 36
    assert max(k[".sgpr_count"] for k in in_order) <= 76
