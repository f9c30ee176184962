"""LDS of the compositing kernels: a slot per wave that is launched, not a
fixed number of them (a workgroup of one 64-pixel wave with four waves' LDS
leaves most of a CU empty).  Read from the metadata of the built library's
code objects."""
import os
import struct

import pytest

msgpack = pytest.importorskip("msgpack")

LIB = os.path.join(os.path.dirname(os.path.abspath(__file__)), "..", "paper_2511_22793_amd", "libgsparc.so")
EM_AMDGPU, NT_AMDGPU_METADATA = 224, 32


def _kernels():
    """{mangled name: metadata} of every kernel in the library."""
    data, out, at = open(LIB, "rb").read(), {}, 1
    while True:
        at = data.find(b"\x7fELF", at)
        if at < 0:
            return out
        if struct.unpack_from("<H", data, at + 18)[0] == EM_AMDGPU:
            phoff, = struct.unpack_from("<Q", data, at + 32)
            phsize, phnum = struct.unpack_from("<HH", data, at + 54)
            for k in range(phnum):
                h = at + phoff + k * phsize
                kind, = struct.unpack_from("<I", data, h)
                off, = struct.unpack_from("<Q", data, h + 8)
                if kind == 4:  # a note: name size, data size, type
                    n, d, t = struct.unpack_from("<III", data, at + off)
                    if t == NT_AMDGPU_METADATA:
                        start = at + off + 12 + (n + 3) // 4 * 4
                        meta = msgpack.unpackb(data[start:start + d], strict_map_key=False)
                        out.update((x[".name"], x) for x in meta["amdhsa.kernels"])
        at += 4


@pytest.mark.skipif(not os.path.exists(LIB), reason="the library is not built")
def test_compositing_kernels_have_no_fixed_wave_slots():
    kernels = {n: m for n, m in _kernels().items()
               if any(k in n for k in ("7k_blendI", "10k_blend_mxI", "15k_blend_mx_longI", "15k_blend_persist"))}
    assert len(kernels) >= 16
    fixed = {n: m[".group_segment_fixed_size"] for n, m in kernels.items()}
    assert max(fixed.values()) <= 64, fixed
