"""The device code in the built library: no kernel needs scratch memory, which the runtime
would allocate at its first launch (the entry points allocate nothing)."""
import struct

import pytest

B = pytest.importorskip("paper_2606_13126_amd._binding")

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects():
    """The gfx950 ELF images of the library's offload bundles."""
    blob = open(B.LIB_PATH, "rb").read()
    at = blob.find(MAGIC)
    while at >= 0:
        n, = struct.unpack_from("<Q", blob, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(n):
            off, size, id_len = struct.unpack_from("<QQQ", blob, p)
            name = blob[p + 24:p + 24 + id_len]
            p += 24 + id_len
            if b"gfx950" in name and size:
                yield blob[at + off:at + off + size]
        at = blob.find(MAGIC, at + 1)


def private_bytes(elf):
    """Private segment bytes per lane of every kernel (the second word of its descriptor)."""
    shoff, = struct.unpack_from("<Q", elf, 40)
    shentsize, shnum = struct.unpack_from("<HH", elf, 58)
    secs = [struct.unpack_from("<IIQQQQIIQQ", elf, shoff + i * shentsize) for i in range(shnum)]
    out = {}
    for name, kind, flags, addr, off, size, link, info, align, entsize in secs:
        if kind != 11:   # SHT_DYNSYM
            continue
        strs = secs[link]
        for s in range(off, off + size, entsize):
            st_name, st_info, st_other, shndx, value, st_size = struct.unpack_from("<IBBHQQ", elf, s)
            end = elf.index(b"\0", strs[4] + st_name)
            sym = elf[strs[4] + st_name:end].decode()
            if sym.endswith(".kd") and 0 < shndx < shnum:
                at = secs[shndx][4] + value - secs[shndx][3]
                out[sym[:-3]] = struct.unpack_from("<I", elf, at + 4)[0]
    return out


def test_no_kernel_uses_scratch():
    kernels = {}
    for elf in code_objects():
        kernels.update(private_bytes(elf))
    assert len(kernels) > 50
    assert {k: v for k, v in kernels.items() if v} == {}
