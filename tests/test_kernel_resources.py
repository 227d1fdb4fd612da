"""The built library's code objects, read on the host: kernels whose operand
rings must stay in registers use no scratch memory."""
import struct

import pytest

from paper_2609_28358_amd import mxconv as mx

msgpack = pytest.importorskip("msgpack")
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"
SHT_NOTE = 7


def _kernels():
    """The metadata of every gfx950 kernel in the library."""
    mx.lib()
    data = open(mx.LIB_PATH, "rb").read()
    out = []
    at = data.find(MAGIC)
    while at >= 0:
        n, = struct.unpack_from("<Q", data, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(n):
            off, size, tlen = struct.unpack_from("<QQQ", data, p)
            triple = data[p + 24:p + 24 + tlen]
            p += 24 + tlen
            if size and b"gfx950" in triple:
                out += _metadata(data[at + off:at + off + size])
        at = data.find(MAGIC, at + 1)
    return out


def _metadata(elf):
    shoff, = struct.unpack_from("<Q", elf, 0x28)
    shsize, shnum = struct.unpack_from("<HH", elf, 0x3A)
    for i in range(shnum):
        kind, = struct.unpack_from("<I", elf, shoff + i * shsize + 4)
        off, size = struct.unpack_from("<QQ", elf, shoff + i * shsize + 0x18)
        end = off + size
        while kind == SHT_NOTE and off < end:
            nlen, dlen, typ = struct.unpack_from("<III", elf, off)
            name = off + 12
            desc = name + (nlen + 3) // 4 * 4
            if elf[name:name + 6] == b"AMDGPU" and typ == 32:
                return msgpack.unpackb(elf[desc:desc + dlen], strict_map_key=False)["amdhsa.kernels"]
            off = desc + (dlen + 3) // 4 * 4
    return []


@pytest.mark.parametrize("name,count", [("wgrad_row_kernel", 13)])
def test_no_scratch(name, count):
    found = {k[".symbol"]: k[".private_segment_fixed_size"] for k in _kernels() if name in k[".name"]}
    assert len(found) == count
    assert not {k: v for k, v in found.items() if v}
