"""Registers and stack of the built kernels, read from the library's own code objects (no GPU): what a change of the source
can lose without any result changing.  A SIMD has 512 registers per lane for its wavefronts."""
import functools
import struct

import msgpack
import pytest

from paper_2605_25451_amd import build

GENERIC = "attn_%s_generic_kernelI%sLi%dELb%dE"


def code_objects(blob):
    at = blob.find(b"__CLANG_OFFLOAD_BUNDLE__")
    while at >= 0:
        count, = struct.unpack_from("<Q", blob, at + 24)
        p = at + 32
        for _ in range(count):
            offset, size, name_len = struct.unpack_from("<QQQ", blob, p)
            if b"gfx950" in blob[p + 24:p + 24 + name_len] and size:
                yield blob[at + offset:at + offset + size]
            p += 24 + name_len
        at = blob.find(b"__CLANG_OFFLOAD_BUNDLE__", at + 24)


def metadata(elf):
    """The kernels' entries of the AMDGPU metadata note (type 32)."""
    sections, = struct.unpack_from("<Q", elf, 0x28)
    entry, count = struct.unpack_from("<HH", elf, 0x3A)
    for i in range(count):
        kind, = struct.unpack_from("<I", elf, sections + i * entry + 4)
        if kind != 7:                                        # SHT_NOTE
            continue
        p, size = struct.unpack_from("<QQ", elf, sections + i * entry + 24)
        end = p + size
        while p < end:
            name, desc, note = struct.unpack_from("<III", elf, p)
            body = p + 12 + (name + 3) // 4 * 4
            if note == 32:
                yield from msgpack.unpackb(elf[body:body + desc], strict_map_key=False).get("amdhsa.kernels", [])
            p = body + (desc + 3) // 4 * 4


def functions(elf):
    """Names of the functions in the symbol table."""
    sections, = struct.unpack_from("<Q", elf, 0x28)
    entry, count = struct.unpack_from("<HH", elf, 0x3A)
    heads = [struct.unpack_from("<IIQQQQIIQQ", elf, sections + i * entry) for i in range(count)]
    found = set()
    for _, kind, _, _, offset, size, link, _, _, step in heads:
        if kind == 2:                                        # SHT_SYMTAB
            strings = heads[link][4]
            for p in range(offset, offset + size, step):
                name, info = struct.unpack_from("<IB", elf, p)
                if info & 15 == 2:                           # STT_FUNC
                    found.add(elf[strings + name:elf.index(b"\0", strings + name)])
    return found


@functools.lru_cache(None)
def kernels():
    with open(build.LIB, "rb") as f:
        blob = f.read()
    found = {k[".name"]: k for elf in code_objects(blob) for k in metadata(elf)}
    assert len(found) > 200
    return found


def registers(part):
    got = [k[".vgpr_count"] for n, k in kernels().items() if part in n]
    assert got, part
    return max(got)


def test_kernels_call_no_function():
    """What several kernels share is inlined: a call holds the registers of the largest caller and moves its rows through
    the stack."""
    with open(build.LIB, "rb") as f:
        blob = f.read()
    for elf in code_objects(blob):
        names = {n.encode() for k in metadata(elf) for n in (k[".name"],)}
        assert functions(elf) <= names, functions(elf) - names


@pytest.mark.parametrize("storage", ["f", "DF16b"])
@pytest.mark.parametrize("causal", [0, 1])
def test_dq_of_head_size_32_keeps_two_wavefronts_per_simd(storage, causal):
    assert registers(GENERIC % ("dq", storage, 32, causal) + "Li8E") <= 256


@pytest.mark.parametrize("storage", ["f", "DF16b"])
@pytest.mark.parametrize("causal", [0, 1])
def test_attention_of_head_size_72_keeps_two_wavefronts_per_simd(storage, causal):
    assert registers(GENERIC % ("fwd", storage, 72, causal)) <= 256
