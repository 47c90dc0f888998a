"""Where the decoder lies in the built library's gfx950 code object (no GPU
needed): its speed depends on that by up to 13 %, and the size of any other
kernel in the file moves it."""
import os
import struct

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2606_18900_amd", "liblz.so")
AMDGPU = 224                                       # e_machine


def _functions(elf):
    """(name, address) of the function symbols of an ELF64 image."""
    shoff, = struct.unpack_from("<Q", elf, 40)
    entsize, num, = struct.unpack_from("<HH", elf, 58)
    sec = [struct.unpack_from("<IIQQQQIIQQ", elf, shoff + entsize * k) for k in range(num)]
    for _, kind, _, _, off, size, link, _, _, ent in sec:
        if kind != 2:                              # SHT_SYMTAB
            continue
        names = sec[link][4]
        for o in range(off, off + size, ent):
            name, info, _, _, value, _ = struct.unpack_from("<IBBHQQ", elf, o)
            if info & 15 == 2:                     # STT_FUNC
                end = elf.index(b"\0", names + name)
                yield elf[names + name:end].decode(), value


def test_decoder_begins_where_it_is_fastest():
    if not os.path.exists(LIB):
        pytest.skip("liblz.so is not built")
    data, at = open(LIB, "rb").read(), []
    o = data.find(b"\x7fELF", 4)
    while o >= 0:
        if struct.unpack_from("<H", data, o + 18)[0] == AMDGPU:
            at += [a for n, a in _functions(data[o:]) if "k_decodeILj1E" in n]
        o = data.find(b"\x7fELF", o + 4)
    assert len(at) == 1
    assert at[0] % 0x1000 == 0xe00 and 0x17e00 <= at[0] <= 0x1ee00, hex(at[0])
