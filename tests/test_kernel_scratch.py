"""Register spills of the built kernels, read from the metadata of the code
objects in libsparse_linear.so: no kernel instance that the library's choice of
kernel and shape can reach may use scratch memory (a spilled register is
reloaded in every epilogue or window loop).
"""
import os
import struct

import msgpack
import pytest

import paper_2211_07715_amd as sl

MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def _code_objects(data):
    at = data.find(MAGIC)
    while at >= 0:
        n, = struct.unpack_from("<Q", data, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(n):
            off, size, idlen = struct.unpack_from("<QQQ", data, p)
            name = data[p + 24:p + 24 + idlen].decode()
            p += 24 + idlen
            if "gfx950" in name and size:
                yield data[at + off:at + off + size]
        at = data.find(MAGIC, at + len(MAGIC))


def _metadata(elf):
    """The AMDGPU metadata note (type 32) of a 64-bit little-endian ELF."""
    shoff, = struct.unpack_from("<Q", elf, 0x28)
    shentsize, shnum = struct.unpack_from("<HH", elf, 0x3A)
    for i in range(shnum):
        sh = shoff + i * shentsize
        kind, = struct.unpack_from("<I", elf, sh + 4)
        off, size = struct.unpack_from("<QQ", elf, sh + 0x18)
        if kind != 7:  # SHT_NOTE
            continue
        p = off
        while p < off + size:
            namesz, descsz, typ = struct.unpack_from("<III", elf, p)
            desc = p + 12 + (namesz + 3) // 4 * 4
            if typ == 32:
                return msgpack.unpackb(elf[desc:desc + descsz])
            p = desc + (descsz + 3) // 4 * 4
    raise AssertionError("no metadata note")


@pytest.fixture(scope="module")
def kernels():
    if not os.path.exists(sl.LIB_PATH):
        pytest.skip("the library is not built")
    with open(sl.LIB_PATH, "rb") as f:
        data = f.read()
    return {k[".name"]: k for co in _code_objects(data) for k in _metadata(co)["amdhsa.kernels"]}


def test_no_reachable_kernel_spills(kernels):
    for part in ("panel_kernel", "panel_gelu_kernel", "tile_kernel", "split_kernel", "direct_kernel"):
        assert sum(part in n for n in kernels) > 4, part
    # int8 GELU by erf (kind 5) in the 12-wave 8-tile shape, which only SL_PTILE runs
    forced = [n for n in kernels if "sparse_linear_panel_kernelILi5ELi8ELi2ELi12E" in n]
    assert len(forced) == 4
    spilled = {n: k[".private_segment_fixed_size"] for n, k in kernels.items()
               if k[".private_segment_fixed_size"] and n not in forced}
    assert not spilled, spilled
