"""The matmul kernels read their epilogue tables by absolute LDS addresses, counted from the start of their dynamic LDS, which lies behind any
LDS that a kernel declares statically; the FP8 main loop flips bits of such addresses.  So none of them may declare any: checked in the
metadata of the built library, as is that none of them spills to scratch memory.  And the tiles whose fragments do not start where bits
can be flipped must not compile."""
import struct
import subprocess

import msgpack
import pytest

import paper_2303_11257_amd as us
from paper_2303_11257_amd import build

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


def _metadata(key):
    us.lib()                                # there is a built library
    with open(us.library_path(), "rb") as f:
        return {k[".name"]: k[key] for elf in _code_objects(f.read()) for k in _kernels(elf)}


def test_matmul_kernels_have_no_static_lds():
    kernels = _metadata(".group_segment_fixed_size")
    matmul = {n: size for n, size in kernels.items() if "gemm_" in n}
    assert len(matmul) > 100 and any(kernels.values())        # other kernels do have some: the metadata is read
    assert not [n for n, size in matmul.items() if size]


def test_kernels_use_no_scratch():
    kernels = _metadata(".private_segment_fixed_size")
    assert len(kernels) > 100
    assert not [n for n, size in kernels.items() if size]


@pytest.mark.parametrize("a_kc,b_kc,fits", [("true", "true", True), ("true", "false", False), ("false", "true", True)])
def test_fp8_tiles_of_odd_width_are_refused(tmp_path, a_kc, b_kc, fits):
    """FP8 on a tile whose waves are 64 rows by 96 columns: fine while the 96 side is K-contiguous."""
    src = tmp_path / "tile.hip"
    src.write_text('#include "us_gemm_direct.h"\nint bytes = us::DirectTile<us::GemmCfg<256, 192, 4, 2, 128, 2, 1>, true, %s, %s, false>::LDS_BYTES;\n' % (a_kc, b_kc))
    r = subprocess.run([build.HIPCC, *build.FLAGS, "-I", build.CSRC, "--offload-host-only", "-fsyntax-only", str(src)], capture_output=True, text=True)
    assert (r.returncode == 0) == fits and (fits or "a power of two per wave" in r.stderr), r.stderr
