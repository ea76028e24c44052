"""Registers of the built kernels (host only): what the compiler notes beside each of them in the library's code objects.  A vector
register that is spilled in a loop over k tiles is reloaded behind a wait for every load in flight."""
import re
import struct

import pytest

msgpack = pytest.importorskip("msgpack")


def code_objects(blob):
    """gfx950 ELF images of the offload bundles in a shared library"""
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = blob.find(magic)
    while at >= 0:
        count, = struct.unpack_from("<Q", blob, at + len(magic))
        p = at + len(magic) + 8
        for _ in range(count):
            offset, size, n = struct.unpack_from("<QQQ", blob, p)
            if size and b"gfx950" in blob[p + 24:p + 24 + n]:
                yield blob[at + offset:at + offset + size]
            p += 24 + n
        at = blob.find(magic, at + 1)


def kernels(elf):
    """name -> the compiler's note of it (NT_AMDGPU_METADATA, msgpack)"""
    phoff, = struct.unpack_from("<Q", elf, 32)
    size, count = struct.unpack_from("<HH", elf, 54)
    for i in range(count):
        kind, _, offset, _, _, length = struct.unpack_from("<IIQQQQ", elf, phoff + i * size)
        p = offset
        while kind == 4 and p + 12 <= offset + length:
            name, desc, what = struct.unpack_from("<III", elf, p)
            body = p + 12 + (name + 3) // 4 * 4
            if what == 32:
                for k in msgpack.unpackb(elf[body:body + desc])["amdhsa.kernels"]:
                    yield k[".name"], k
            p = body + (desc + 3) // 4 * 4


@pytest.fixture(scope="module")
def notes():
    from paper_1807_11205_amd import api
    api.lib()
    with open(api.LIB_PATH, "rb") as f:
        blob = f.read()
    found = {name: k for elf in code_objects(blob) for name, k in kernels(elf)}
    assert len(found) > 100
    return found


@pytest.mark.parametrize("kernel, variants", [("f32_window_kernel", 8), ("lars_reduce_groups", 2), ("lars_update", 6), ("lars_begin", 1)])
def test_vector_registers_are_not_spilled(notes, kernel, variants):
    of = {n: k for n, k in notes.items() if re.search(r"\d" + kernel + r"(I|E|P)", n)}
    assert len(of) == variants, sorted(of)
    assert not {n: k[".vgpr_spill_count"] for n, k in of.items() if k[".vgpr_spill_count"]}
