"""What the compiler made of the kernels, from the metadata of the built library's code object:
a kernel with scratch memory but no spilled registers keeps an array there that it indexes with
a variable, two memory round trips for every access in its inner loop."""
import os
import struct

import msgpack
import pytest

import paper_2606_10896_amd as gmm

LIB = os.path.join(os.path.dirname(gmm.__file__), "libflashgmm.so")


def _code_objects(blob):
    """The gfx950 images of the library's offload bundles."""
    magic, i = b"__CLANG_OFFLOAD_BUNDLE__", -1
    while (i := blob.find(magic, i + 1)) >= 0:
        (count,) = struct.unpack_from("<Q", blob, i + 24)
        o = i + 32
        for _ in range(count):
            off, size, length = struct.unpack_from("<QQQ", blob, o)
            if b"gfx950" in blob[o + 24:o + 24 + length]:
                yield blob[i + off:i + off + size]
            o += 24 + length


def _kernels(path):
    """The kernels' metadata (the msgpack note of every image)."""
    with open(path, "rb") as f:
        blob = f.read()
    for elf in _code_objects(blob):
        (shoff,) = struct.unpack_from("<Q", elf, 40)
        shsize, shnum = struct.unpack_from("<HH", elf, 58)
        for s in range(shnum):
            h = shoff + s * shsize
            if struct.unpack_from("<I", elf, h + 4)[0] != 7:          # SHT_NOTE
                continue
            p, size = struct.unpack_from("<QQ", elf, h + 24)
            end = p + size
            while p < end:
                nlen, dlen, kind = struct.unpack_from("<III", elf, p)
                p += 12 + (nlen + 3 & ~3)
                if kind == 32:                                          # NT_AMDGPU_METADATA
                    yield from msgpack.unpackb(elf[p:p + dlen])["amdhsa.kernels"]
                p += dlen + 3 & ~3


@pytest.fixture(scope="module")
def kernels():
    gmm.load_library()
    return {k[".name"]: k for k in _kernels(LIB)}


def test_every_width_has_its_screening_kernels(kernels):
    for d in (64, 128, 192, 256, 384, 512, 640, 768, 896, 1024):
        for iso in (0, 1):
            for split in (0, 1):
                assert any(f"k_coarseILi{d}ELb{iso}ELb{split}E" in n for n in kernels), d


def test_no_kernel_keeps_an_array_in_scratch_memory(kernels):
    bad = {n: k[".private_segment_fixed_size"] for n, k in kernels.items()
           if k[".private_segment_fixed_size"] > 0 and k[".vgpr_spill_count"] == 0}
    assert not bad, bad
