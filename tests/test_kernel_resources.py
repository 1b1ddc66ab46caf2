"""Registers of the built pack kernels, read from the metadata of libspin.so's own gfx950 code objects: the waves per SIMD that a
kernel of one side reaches by itself must not be lost to what another side needs (a SIMD has 512 registers per lane)."""
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
@pytest.mark.parametrize("np,ring,side,most", [(2, "o", "left", 256),      # two waves; with the right pack in one kernel: one
                                               (1, "o", "right", 168),     # three; two
                                               (2, "m", "right", 168),     # three; two
                                               (7, "j", "right", 256)])    # two; one
def test_one_sided_packs_keep_their_waves(np, ring, side, most):
    which = {"both": 0, "left": 1, "right": 2}[side]
    found = {n: v for n, (v, _) in kernels().items()
             if re.search(r"pack_kernelILi%dE%sLb[01]ELb0ELb[01]ELNS\w*PackSideE%dE" % (np, ring, which), n)}
    assert len(found) >= 2 and max(found.values()) <= most, found


def test_packs_of_three_parties_keep_two_waves():
    found = {n: v for n, (v, _) in kernels().items() if re.search(r"pack_(grouped_)?kernelILi3E(m|LNS)", n)}
    assert len(found) >= 5 and max(found.values()) <= 256, found


def test_grouped_packs_of_right_operands_for_eight_parties():
    spilled = [s for n, (_, s) in kernels().items() if re.search(r"pack_grouped_kernelILi8ELNS\w*PackSideE2E", n)]
    assert len(spilled) == 1 and spilled[0] <= 64            # 388 bytes in one kernel with the packs by rows


def test_no_kernel_spills_vector_registers():
    """The compiler can lose a part of a spilled group of registers (wrong words, no error), so no kernel may depend on it."""
    spilled = {n: s for n, (_, s) in kernels().items() if s}
    assert len(kernels()) > 500 and not spilled, spilled
