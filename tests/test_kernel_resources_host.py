"""Scratch memory of the built kernels, read from the code objects in
libpfspec.so (the AMDGPU metadata note of each; no GPU needed).  A lane's
scratch is memory traffic that no launch rule sees."""

import struct

import msgpack
import pytest

from paper_2306_04322_amd import build as B

EM_AMDGPU, SHT_NOTE, NT_AMDGPU_METADATA = 224, 7, 32


def _kernels():
    """{mangled name: metadata} of every kernel in the library."""
    data = open(B.LIB, "rb").read()
    out = {}
    at = data.find(b"\x7fELF", 1)
    while at >= 0:
        if struct.unpack_from("<H", data, at + 18)[0] == EM_AMDGPU:
            shoff, = struct.unpack_from("<Q", data, at + 40)
            shentsize, shnum = struct.unpack_from("<HH", data, at + 58)
            for i in range(shnum):
                sh = at + shoff + i * shentsize
                kind, = struct.unpack_from("<I", data, sh + 4)
                off, size = struct.unpack_from("<QQ", data, sh + 24)
                if kind != SHT_NOTE:
                    continue
                p, end = at + off, at + off + size
                while p < end:
                    namesz, descsz, ntype = struct.unpack_from("<III", data, p)
                    desc = p + 12 + (namesz + 3) // 4 * 4
                    if ntype == NT_AMDGPU_METADATA:
                        meta = msgpack.unpackb(data[desc:desc + descsz], strict_map_key=False)
                        for k in meta["amdhsa.kernels"]:
                            out[k[".name"]] = k
                    p = desc + (descsz + 3) // 4 * 4
        at = data.find(b"\x7fELF", at + 4)
    return out


@pytest.fixture(scope="module")
def kernels():
    k = _kernels()
    assert any("rowpass_kernel" in n for n in k)
    return k


def test_wave_adjoint_stays_in_registers(kernels):
    """The wave-per-transform adjoint row pass: at most 16 registers of a lane
    in scratch, for every row length and order-parameter count."""
    adj = {n: k[".private_segment_fixed_size"] for n, k in kernels.items() if "adjrow_kernel" in n}
    assert len(adj) > 100
    assert {n: b for n, b in adj.items() if b > 64} == {}


def test_register_adjoint_float_rows(kernels):
    """The register form on 4096-point float rows: scratch no larger than with
    the order-parameter count read at run time (eight: 452 bytes)."""
    adj = {n: k[".private_segment_fixed_size"] for n, k in kernels.items() if "adj_row_kernelIfLi4096" in n}
    assert len(adj) == 8
    assert {n: b for n, b in adj.items() if b > 512} == {}
