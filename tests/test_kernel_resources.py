"""Registers of the built kernels, read from the metadata of libspin.so's own gfx950 code objects: the waves per SIMD that the packs
reach (a SIMD has 512 registers per lane), the kernels of one side and those of both, and no spilled registers anywhere."""
import os
import re
import struct

import pytest

msgpack = pytest.importorskip("msgpack")
LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2402_02320_amd", "libspin.so")
EM_AMDGPU, PT_NOTE, NT_AMDGPU_METADATA = 224, 4, 32


def kernels():
    """mangled name -> registers per lane and bytes of spilled ones, of every kernel in the library."""
    blob, out = open(LIB, "rb").read(), {}
    for at in (m.start() for m in re.finditer(b"\x7fELF\x02\x01", blob)):
        if struct.unpack_from("<H", blob, at + 18)[0] != EM_AMDGPU:
            continue
        phoff, = struct.unpack_from("<Q", blob, at + 32)
        size, count = struct.unpack_from("<HH", blob, at + 54)
        for p in range(count):
            kind, _, offset, _, _, filesz = struct.unpack_from("<IIQQQQ", blob, at + phoff + p * size)
            pos, end = at + offset, at + offset + filesz
            while kind == PT_NOTE and pos < end:
                name, desc, note = struct.unpack_from("<III", blob, pos)
                pos += 12 + (name + 3) // 4 * 4
                if note == NT_AMDGPU_METADATA:
                    for k in msgpack.unpackb(blob[pos:pos + desc])["amdhsa.kernels"]:
                        out[k[".name"]] = k[".vgpr_count"], k[".private_segment_fixed_size"]   # AGPRs of the unified file included
                pos += (desc + 3) // 4 * 4
    return out


# mangled ring types: o = unsigned __int128, m = unsigned long, j = unsigned int
@pytest.mark.parametrize("np,ring,side,most", [(2, "o", "left", 256), (2, "o", "both", 256),         # two waves
                                               (1, "o", "right", 168), (1, "o", "both", 168),        # three
                                               (2, "m", "right", 168), (2, "m", "both", 168),        # three
                                               (6, "m", "left", 256), (6, "m", "both", 256),         # two
                                               (7, "j", "right", 256), (8, "j", "both", 168)])       # two, three
def test_packs_keep_their_waves(np, ring, side, most):
    which = {"both": 0, "left": 1, "right": 2}[side]
    found = {n: v for n, (v, _) in kernels().items()
             if re.search(r"pack_kernelILi%dE%sLb[01]ELb0ELb[01]ELNS\w*PackSideE%dE" % (np, ring, which), n)}
    assert len(found) >= (1 if side == "both" else 2) and max(found.values()) <= most, found


@pytest.mark.parametrize("pattern,least,most", [(r"pack_kernelILi3Em", 5, 256), (r"pack_grouped_kernelILi[1-6]E", 6, 256), (r"strassen_pack_kernelILb", 4, 256)])
def test_packs_keep_two_waves(pattern, least, most):
    found = {n: v for n, (v, _) in kernels().items() if re.search(pattern, n)}
    assert len(found) >= least and max(found.values()) <= most, found


def test_no_kernel_spills_vector_registers():
    """The compiler can lose a part of a spilled group of registers (wrong words, no error), so no kernel may depend on it."""
    spilled = {n: s for n, (_, s) in kernels().items() if s}
    assert len(kernels()) > 500 and not spilled, spilled
