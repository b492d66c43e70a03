"""The batched sweep keeps all its values in registers: a spill puts a load, and
with it a wait for every unfinished store, into its walk.  Read from the kernel
descriptions in the built library."""
import os
import struct

import pytest

from paper_1308_1419_amd import tdmap

msgpack = pytest.importorskip("msgpack")

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(blob):
    """The device ELF images of the library's offload bundles."""
    at = blob.find(MAGIC)
    while at >= 0:
        p = at + len(MAGIC)
        (count,) = struct.unpack_from("<Q", blob, p)
        p += 8
        for _ in range(count):
            offset, size, length = struct.unpack_from("<QQQ", blob, p)
            name = blob[p + 24:p + 24 + length]
            p += 24 + length
            if b"gfx950" in name and size:
                yield blob[at + offset:at + offset + size]
        at = blob.find(MAGIC, at + 1)


def _kernels(elf):
    """The entries of amdhsa.kernels in the ELF's AMDGPU metadata note."""
    (shoff,) = struct.unpack_from("<Q", elf, 0x28)
    shentsize, shnum = struct.unpack_from("<HH", elf, 0x3A)
    for i in range(shnum):
        _, kind, _, _, offset, size = struct.unpack_from("<IIQQQQ", elf, shoff + i * shentsize)
        if kind != 7:  # SHT_NOTE
            continue
        end = offset + size
        while offset < end:
            namesz, descsz, note = struct.unpack_from("<III", elf, offset)
            desc = offset + 12 + (namesz + 3) // 4 * 4
            if note == 32 and elf[offset + 12:offset + 18] == b"AMDGPU":
                yield from msgpack.unpackb(elf[desc:desc + descsz])["amdhsa.kernels"]
            offset = desc + (descsz + 3) // 4 * 4


def test_batched_sweep_has_no_scratch():
    if not os.path.exists(tdmap.LIB_PATH):
        pytest.skip("the library is not built")
    with open(tdmap.LIB_PATH, "rb") as f:
        blob = f.read()
    scratch = {k[".name"]: k[".private_segment_fixed_size"]
               for elf in _code_objects(blob) for k in _kernels(elf)
               if "edm_batched_sweep_kernel" in k[".name"]}
    assert len(scratch) == 4
    assert set(scratch.values()) == {0}, scratch
