"""Registers of the kernels as built, from the code object's own metadata: the decode-shaped kernel fits a compute unit eight
times (64 vector registers), and nothing spills."""
import os
import struct

import pytest

msgpack = pytest.importorskip("msgpack")
SO = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2605_11093_amd", "libdmi.so")


def _code_objects(blob):
    """The ELF images for the GPU in the library's offload bundles."""
    magic, at = b"__CLANG_OFFLOAD_BUNDLE__", 0
    while (at := blob.find(magic, at)) >= 0:
        (n,) = struct.unpack_from("<Q", blob, at + 24)
        p = at + 32
        for _ in range(n):
            off, size, length = struct.unpack_from("<QQQ", blob, p)
            name = blob[p + 24:p + 24 + length].decode()
            p += 24 + length
            if "gfx950" in name and size:
                yield blob[at + off:at + off + size]
        at += len(magic)


def _kernels(elf):
    shoff, = struct.unpack_from("<Q", elf, 0x28)
    size, count = struct.unpack_from("<HH", elf, 0x3A)
    for i in range(count):
        kind, = struct.unpack_from("<I", elf, shoff + i * size + 4)
        off, length = struct.unpack_from("<QQ", elf, shoff + i * size + 24)
        if kind != 7:                                   # notes
            continue
        while length >= 12:
            n_name, n_desc, what = struct.unpack_from("<III", elf, off)
            desc = off + 12 + (n_name + 3) // 4 * 4
            if what == 32:                              # AMDGPU metadata
                yield from msgpack.unpackb(elf[desc:desc + n_desc], strict_map_key=False)["amdhsa.kernels"]
            step = desc + (n_desc + 3) // 4 * 4 - off
            off, length = off + step, length - step


@pytest.fixture(scope="module")
def kernels():
    if not os.path.exists(SO):
        pytest.skip("the library has not been built")
    with open(SO, "rb") as f:
        found = [k for e in _code_objects(f.read()) for k in _kernels(e)]
    assert found
    return {k[".name"]: k for k in found}


def test_nothing_spills(kernels):
    assert not [n for n, k in kernels.items() if k[".private_segment_fixed_size"] or k.get(".vgpr_spill_count")]


def test_the_decode_shaped_kernel_fits_eight_times(kernels):
    decode = {n: k[".vgpr_count"] for n, k in kernels.items() if "capture_decode_kernel" in n}
    assert len(decode) >= 16
    assert not {n: v for n, v in decode.items() if v > 64}
