"""The GPU code in the built library, from its ELF headers and kernel metadata
alone (no GPU needed): no kernel keeps registers or arrays in private memory,
and the constant tables are reached directly, not through an address table."""

import struct

import pytest

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects():
    from paper_1902_05320_amd import build
    with open(build.LIB_PATH, "rb") as f:
        blob = f.read()
    at = blob.find(MAGIC)
    while at >= 0:
        (count,) = struct.unpack_from("<Q", blob, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(count):
            off, size, tlen = struct.unpack_from("<QQQ", blob, p)
            triple = blob[p + 24:p + 24 + tlen]
            p += 24 + tlen
            if b"gfx950" in triple and size:
                yield blob[at + off:at + off + size]
        at = blob.find(MAGIC, p)


def _sections(elf):
    """(name, type, offset, size) of each section."""
    (shoff,) = struct.unpack_from("<Q", elf, 40)
    num, names = struct.unpack_from("<HH", elf, 60)
    raw = [struct.unpack_from("<IIQQQQ", elf, shoff + 64 * k) for k in range(num)]
    base = raw[names][4]
    return [(elf[base + r[0]:elf.index(b"\0", base + r[0])].decode(), r[1], r[4], r[5]) for r in raw]


def _kernels():
    msgpack = pytest.importorskip("msgpack")
    out = {}
    for elf in _code_objects():
        for name, kind, off, size in _sections(elf):
            if kind != 7:  # SHT_NOTE
                continue
            nsz, dsz, ntype = struct.unpack_from("<III", elf, off)
            if ntype != 32:  # NT_AMDGPU_METADATA
                continue
            desc = off + 12 + (nsz + 3) // 4 * 4
            for k in msgpack.unpackb(elf[desc:desc + dsz])["amdhsa.kernels"]:
                out[k[".name"]] = k
    return out


def test_no_kernel_uses_private_memory():
    # (private memory is allocated by the runtime at a kernel's first launch,
    # and an array in it is a round trip to memory in the middle of a chain)
    kernels = _kernels()
    assert len(kernels) > 60
    bad = {n: k[".private_segment_fixed_size"] for n, k in kernels.items()
           if k[".private_segment_fixed_size"] or k.get(".vgpr_spill_count")}
    assert not bad, bad


def test_constant_tables_are_reached_directly():
    # a table that the loader can see costs each use a load of its address from
    # the offset table; only the static workspace has to be seen
    for elf in _code_objects():
        sec = {name: (off, size) for name, _, off, size in _sections(elf)}
        off, size = sec[".dynsym"]
        strs = sec[".dynstr"][0]
        for k in range(size // 24):
            name, info = struct.unpack_from("<IB", elf, off + 24 * k)
            if info & 15 == 1:  # STT_OBJECT
                sym = elf[strs + name:elf.index(b"\0", strs + name)].decode()
                assert "scratch" in sym or sym.endswith(".kd") or "__hip" in sym, sym
