"""What the compiler made of the kernels whose speed hangs on how many of their wavefronts a SIMD holds: registers and
scratch memory, read from the metadata of the built library (no GPU needed)."""
import os
import re
import struct
import subprocess

import msgpack
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2510_02613_amd", "libelasticmoe.so")


def _sections(elf):
    """(name, type, bytes) of every section of a 64-bit little-endian ELF file."""
    shoff, = struct.unpack_from("<Q", elf, 0x28)
    shentsize, shnum, shstrndx = struct.unpack_from("<HHH", elf, 0x3A)
    raw = [struct.unpack_from("<IIQQQQ", elf, shoff + i * shentsize) for i in range(shnum)]
    names = raw[shstrndx][4]
    for name, kind, _, _, off, size in raw:
        start = names + name
        yield elf[start:elf.index(b"\0", start)].decode(), kind, elf[off:off + size]


def _code_objects(fatbin):
    """The gfx950 images of the offload bundles in a .hip_fatbin section, one bundle per source file."""
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = fatbin.find(magic)
    while at >= 0:
        count, = struct.unpack_from("<Q", fatbin, at + len(magic))
        pos = at + len(magic) + 8
        for _ in range(count):
            off, size, idlen = struct.unpack_from("<QQQ", fatbin, pos)
            if b"gfx950" in fatbin[pos + 24:pos + 24 + idlen] and size:
                yield fatbin[at + off:at + off + size]
            pos += 24 + idlen
        at = fatbin.find(magic, at + len(magic))


@pytest.fixture(scope="module")
def kernels():
    """"k_name<template arguments>" -> metadata, of every kernel of the library."""
    assert os.path.exists(LIB), "the library is not built"
    with open(LIB, "rb") as f:
        fatbin = next(data for name, _, data in _sections(f.read()) if name == ".hip_fatbin")
    found = {}
    for image in _code_objects(fatbin):
        for _, kind, notes in _sections(image):
            pos = 0
            while kind == 7 and pos + 12 <= len(notes):           # SHT_NOTE
                namesz, descsz, what = struct.unpack_from("<III", notes, pos)
                desc = pos + 12 + (namesz + 3 & ~3)
                if what == 32:                                     # the AMDGPU metadata
                    for k in msgpack.unpackb(notes[desc:desc + descsz])["amdhsa.kernels"]:
                        found[k[".name"]] = k
                pos = desc + (descsz + 3 & ~3)
    plain = subprocess.run(["c++filt"], input="\n".join(found), capture_output=True, text=True, check=True).stdout.split("\n")
    return {re.sub(r"\(anonymous namespace\)::|emoe::|^void ", "", p).split("(")[0]: k for p, k in zip(plain, found.values())}


def _waves(kernel):
    """Wavefronts per SIMD that the registers leave room for: 512 of them, in granules of 8."""
    return min(8, 512 // (kernel[".vgpr_count"] + 7 & ~7))


@pytest.mark.parametrize("pattern,waves", [
    (r"k_expert_decode<true, (true|false), 0(, .*)?>", 4), (r"k_expert_decode<false, false, 0>", 4),   # short contractions
    (r"k_expert_decode<true, true, 1(, .*)?>", 3), (r"k_expert_decode<true, (true|false), 2(, .*)?>", 2),
    (r"k_expert_f32_tile<.*>", 7),
    (r"k_expert_ring<.*>", 2), (r"k_expert_gemm_mfma8<.*>", 2),
])
def test_wavefronts_per_simd(kernels, pattern, waves):
    """As many wavefronts as the comment at the kernel says fit beside each other (a kernel whose code asks for fewer may have room for more), none by way of scratch memory."""
    mine = {n: k for n, k in kernels.items() if re.fullmatch(pattern, n)}
    assert mine
    for name, k in mine.items():
        assert _waves(k) >= waves, (name, k[".vgpr_count"])
        assert k[".private_segment_fixed_size"] == 0 and k[".vgpr_spill_count"] == 0, name


def test_scalar_spills_of_the_ring_kernels(kernels):
    """Kernels that read the tile list (GEMM-2, and GEMM-1 of routed passes, of more than 1024 tokens or 256 slots) hold nothing of the code that derives tiles: no scalar
    is spilled, GEMM-1 needs the registers that GEMM-2 needs.  That code's own spills lie in front of its K loops."""
    mine = {n: k for n, k in kernels.items() if n.startswith("k_expert_ring<")}
    for tiles in (1, 2):
        first, second = mine.pop(f"k_expert_ring<true, false, {tiles}, TileList>"), mine.pop(f"k_expert_ring<false, false, {tiles}>")
        assert first[".sgpr_spill_count"] == second[".sgpr_spill_count"] == 0
        assert first[".vgpr_count"] <= second[".vgpr_count"]
    for name, k in mine.items():
        assert k[".sgpr_spill_count"] <= (56 if name in ("k_expert_ring<true, false, 1>", "k_expert_ring<true, false, 2>") else 0), name
