"""The channel kernels read their LDS window by absolute address, from 0 on (ttcf_channel.hip): that
holds as long as nothing they call declares LDS of a fixed size, which would come first. The built
library's own kernel descriptions say so."""
import os
import struct

import msgpack
import pytest

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2312_02990_amd",
                   "libttcf.so")


def kernels(blob):
    """Kernel descriptions (dicts) of every gfx950 code object in the library's offload bundles."""
    magic, at = b"__CLANG_OFFLOAD_BUNDLE__", 0
    while (at := blob.find(magic, at)) >= 0:
        count, = struct.unpack_from("<Q", blob, at + 24)
        entry = at + 32
        for _ in range(count):
            offset, size, name_len = struct.unpack_from("<QQQ", blob, entry)
            name = blob[entry + 24:entry + 24 + name_len]
            entry += 24 + name_len
            if b"gfx950" in name and size:
                yield from notes(blob[at + offset:at + offset + size])
        at += len(magic)


def notes(elf):
    phoff, = struct.unpack_from("<Q", elf, 32)
    phsize, phnum = struct.unpack_from("<HH", elf, 54)
    for k in range(phnum):
        kind, _, offset, _, _, size = struct.unpack_from("<IIQQQQ", elf, phoff + k * phsize)
        end = offset + size
        while kind == 4 and offset + 12 <= end:  # PT_NOTE
            name, desc, note = struct.unpack_from("<III", elf, offset)
            body = offset + 12 + (name + 3) // 4 * 4
            if note == 32:  # AMDGPU metadata
                yield from msgpack.unpackb(elf[body:body + desc])["amdhsa.kernels"]
            offset = body + (desc + 3) // 4 * 4


def test_no_fixed_lds_before_the_window():
    if not os.path.exists(LIB):
        pytest.skip("library not built")
    with open(LIB, "rb") as f:
        found = {k[".name"]: k[".group_segment_fixed_size"] for k in kernels(f.read())}
    window = {n: v for n, v in found.items() if "13ChannelLaunch" in n}  # (their argument)
    assert len(window) == 2, sorted(n for n in found if "k_channel" in n)
    assert set(window.values()) == {0}
