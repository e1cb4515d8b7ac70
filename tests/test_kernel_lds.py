"""The matmul kernels read their epilogue tables by absolute LDS addresses, counted from the start of their dynamic LDS, which lies behind any
LDS that a kernel declares statically.  So none of them may declare any: checked in the metadata of the built library."""
import struct

import msgpack

import paper_2303_11257_amd as us

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(data):
    at = data.find(MAGIC)
    while at >= 0:
        pos = at + len(MAGIC)
        count, = struct.unpack_from("<Q", data, pos)
        pos += 8
        for _ in range(count):
            offset, size, length = struct.unpack_from("<QQQ", data, pos)
            triple = data[pos + 24:pos + 24 + length]
            pos += 24 + length
            if size and b"amdgcn" in triple:
                yield data[at + offset:at + offset + size]
        at = data.find(MAGIC, at + 1)


def _kernels(elf):
    """The kernels' entries of an ELF file's AMDGPU metadata note (note type 32, MessagePack)."""
    shoff, = struct.unpack_from("<Q", elf, 40)
    shentsize, shnum = struct.unpack_from("<HH", elf, 58)
    for s in range(shnum):
        kind, = struct.unpack_from("<I", elf, shoff + s * shentsize + 4)
        offset, size = struct.unpack_from("<QQ", elf, shoff + s * shentsize + 24)
        if kind != 7:                       # SHT_NOTE
            continue
        end = offset + size
        while offset < end:
            name, desc, note = struct.unpack_from("<III", elf, offset)
            offset += 12 + (name + 3) // 4 * 4
            if note == 32:
                yield from msgpack.unpackb(elf[offset:offset + desc], raw=False)["amdhsa.kernels"]
            offset += (desc + 3) // 4 * 4


def test_matmul_kernels_have_no_static_lds():
    us.lib()                                # there is a built library
    with open(us.library_path(), "rb") as f:
        kernels = {k[".name"]: k[".group_segment_fixed_size"] for elf in _code_objects(f.read()) for k in _kernels(elf)}
    matmul = {n: size for n, size in kernels.items() if "gemm_" in n}
    assert len(matmul) > 100 and any(kernels.values())        # other kernels do have some: the metadata is read
    assert not [n for n, size in matmul.items() if size]
