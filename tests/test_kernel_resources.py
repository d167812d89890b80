"""Scratch memory of the built kernels, from the metadata of libtnc.so's own
code objects: sums that are meant to live in registers do."""
import re
import struct

import pytest

from paper_2608_13110_amd import LIB_PATH

msgpack = pytest.importorskip("msgpack")


def code_objects():
    """The gfx950 ELF images in the library's offload bundles."""
    blob = open(LIB_PATH, "rb").read()
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    for m in re.finditer(magic, blob):
        at = m.start() + len(magic)
        (count,) = struct.unpack_from("<Q", blob, at)
        if count > 8:  # the magic as a string of the runtime's, not a bundle
            continue
        at += 8
        for _ in range(count):
            off, size, ident = struct.unpack_from("<QQQ", blob, at)
            name = blob[at + 24:at + 24 + ident]
            at += 24 + ident
            if b"gfx950" in name and size:
                yield blob[m.start() + off:m.start() + off + size]


def kernels():
    """{kernel symbol: metadata} over all code objects."""
    found = {}
    for elf in code_objects():
        shoff, = struct.unpack_from("<Q", elf, 40)
        entsize, num = struct.unpack_from("<HH", elf, 58)
        for i in range(num):
            kind, = struct.unpack_from("<I", elf, shoff + i * entsize + 4)
            off, size = struct.unpack_from("<QQ", elf, shoff + i * entsize + 24)
            if kind != 7:  # SHT_NOTE
                continue
            namesz, descsz, ntype = struct.unpack_from("<III", elf, off)
            if ntype == 32:  # NT_AMDGPU_METADATA
                desc = elf[off + 12 + (namesz + 3) // 4 * 4:][:descsz]
                for k in msgpack.unpackb(desc, strict_map_key=False)["amdhsa.kernels"]:
                    found[k[".name"]] = k
    return found


def test_join_sums_stay_in_registers():
    late = {n: k for n, k in kernels().items() if "k_late_dot" in n}
    assert len(late) >= 16  # four tensor types, one to eight columns
    assert {n: k[".private_segment_fixed_size"] for n, k in late.items() if k[".private_segment_fixed_size"]} == {}


def test_complex64_passes_stay_in_registers():
    passes = {n: k for n, k in kernels().items() if re.search(r"k_pass(_g)?ILi\dELb[01]ELb[01]ELi\d+ELi0E", n)}
    assert len(passes) >= 30  # 2 to 32 entries per thread, whole tiles and several per block
    assert {n: k[".private_segment_fixed_size"] for n, k in passes.items() if k[".private_segment_fixed_size"]} == {}
    # eight entries per thread, several tiles per block: seven waves per SIMD (512 / 7 registers)
    small = {n: k[".vgpr_count"] for n, k in passes.items() if re.search(r"ILi3ELb1ELb0E", n)}
    assert small and max(small.values()) <= 72, small
