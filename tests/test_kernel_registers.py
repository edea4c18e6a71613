"""Registers of the built kernels, from the metadata notes of the library's
code objects (host side, no GPU).

The compiler pairs LDS stores of neighbouring rows (ds_write2_b32, offsets in
elements).  Where some of the values are in accumulation registers and some are
not, it has divided a byte offset twice: the columns kernel of FP32 n = 8,
compiled with accumulation registers, stores rows 4 and 5 of a plane with
`ds_write2_b32 .. offset0:8 offset1:40`, where row 4 is at element 32 (byte 128,
128 / 4 / 4 = 8).  The kernels that write columns to LDS therefore use none."""
import os
import struct

import pytest

import paper_1304_7054_amd as kron

msgpack = pytest.importorskip("msgpack")

COLUMNS = ("kron3d_cols_kernel", "kron_grouped_f32_kernel", "kron_backward_kernel", "kron_backward_grouped_kernel",
           "kron_strided_cols_kernel", "kron_nd_fused_kernel")
EM_AMDGPU, SHT_NOTE, NT_AMDGPU_METADATA = 224, 7, 32


def _kernels():
    """The metadata of every kernel in the library."""
    with open(kron._binding.LIB_PATH, "rb") as f:
        data = f.read()
    at = data.find(b"\x7fELF", 4)
    while at >= 0:
        machine = struct.unpack_from("<H", data, at + 18)[0]
        if machine == EM_AMDGPU:
            shoff = struct.unpack_from("<Q", data, at + 40)[0]
            size, count = struct.unpack_from("<HH", data, at + 58)
            for i in range(count):
                kind, = struct.unpack_from("<I", data, at + shoff + i * size + 4)
                off, length = struct.unpack_from("<QQ", data, at + shoff + i * size + 24)
                if kind != SHT_NOTE:
                    continue
                pos, end = at + off, at + off + length
                while pos < end:
                    name, desc, note = struct.unpack_from("<III", data, pos)
                    body = pos + 12 + (name + 3) // 4 * 4
                    if note == NT_AMDGPU_METADATA:
                        yield from msgpack.unpackb(data[body:body + desc])["amdhsa.kernels"]
                    pos = body + (desc + 3) // 4 * 4
        at = data.find(b"\x7fELF", at + 4)


def test_column_kernels_use_no_accumulation_registers():
    if not os.path.exists(kron._binding.LIB_PATH):
        pytest.skip("the library is not built")
    seen = {k: 0 for k in COLUMNS}
    for kernel in _kernels():
        name = kernel[".name"]
        for k in COLUMNS:
            if f"{len(k)}{k}" in name:  # a mangled name's length and identifier
                seen[k] += 1
                assert kernel[".agpr_count"] == 0, name
    assert all(seen.values()), seen
