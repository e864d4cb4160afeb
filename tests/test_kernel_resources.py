"""Scratch memory of the built kernels, from the metadata of the code objects in the library: a function that the compiler does not
inline, or an array that it cannot keep in registers, shows here and costs a kernel up to twice its time."""
import re
import struct

import msgpack

from paper_2508_15212_amd import build


def _code_objects(blob):
    """gfx950 ELF images of the offload bundles in a shared library (one bundle per source file)."""
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    for at in (m.start() for m in re.finditer(magic, blob)):
        (entries,), p = struct.unpack_from("<Q", blob, at + len(magic)), at + len(magic) + 8
        if entries > 16:
            continue
        for _ in range(entries):
            offset, size, id_len = struct.unpack_from("<QQQ", blob, p)
            name = blob[p + 24:p + 24 + id_len]
            p += 24 + id_len
            if b"gfx950" in name and size:
                yield blob[at + offset:at + offset + size]


def _kernels(elf):
    """Entries of amdhsa.kernels: note of type 32, owner AMDGPU."""
    shoff, = struct.unpack_from("<Q", elf, 0x28)
    shentsize, shnum = struct.unpack_from("<HH", elf, 0x3A)
    for i in range(shnum):
        sh = shoff + i * shentsize
        if struct.unpack_from("<I", elf, sh + 4)[0] != 7:       # SHT_NOTE
            continue
        offset, size = struct.unpack_from("<QQ", elf, sh + 24)
        p = offset
        while p + 12 <= offset + size:
            namesz, descsz, kind = struct.unpack_from("<III", elf, p)
            desc = p + 12 + (namesz + 3 & ~3)
            if kind == 32 and elf[p + 12:p + 18] == b"AMDGPU":
                yield from msgpack.unpackb(elf[desc:desc + descsz])["amdhsa.kernels"]
            p = desc + (descsz + 3 & ~3)


def _scratch():
    with open(build.LIB, "rb") as f:
        blob = f.read()
    return {k[".name"]: (k[".private_segment_fixed_size"], bool(k.get(".uses_dynamic_stack", False)))
            for elf in _code_objects(blob) for k in _kernels(elf)}


def test_no_kernel_keeps_its_state_in_scratch():
    found = _scratch()
    assert sum("spark_decode_kernel" in n for n in found) > 100 and sum("spark_prune_kernel" in n for n in found) > 4
    assert not [n for n, (_, dynamic) in found.items() if dynamic]
    # (spilled registers: 388 bytes in top-p decode with sixteen query heads, 156 in the balanced cut with eight and rows of any length)
    assert {n: size for n, (size, _) in found.items() if size > 400} == {}
