"""Registers of the built adjoint kernels, from the code objects' metadata.

A SIMD has 512 registers per lane: a kernel above 256 runs one wave per SIMD, with
nothing to hide its latencies behind.
"""
import re
import struct

import pytest

msgpack = pytest.importorskip("msgpack")


def _kernels():
    from paper_2504_16446_amd._lib import LIB_PATH
    blob = open(LIB_PATH, "rb").read()
    out = {}
    for m in re.finditer(b"AMDGPU\0\0", blob):  # ELF note: name size, descriptor size, type, name, descriptor
        namesz, size, kind = struct.unpack("<III", blob[m.start() - 12:m.start()])
        if namesz == 7 and kind == 32:
            meta = msgpack.unpackb(blob[m.end():m.end() + size])
            out.update({k[".name"]: k for k in meta["amdhsa.kernels"]})
    return out


def test_adjoint_kernels_leave_room_for_two_waves():
    ks = {n: k for n, k in _kernels().items() if "k_backproject" in n}
    assert len(ks) >= 96, len(ks)
    assert {n: k[".vgpr_count"] for n, k in ks.items() if k[".vgpr_count"] > 256} == {}
    # without spilling for it, from 64 coefficients on (a few set-up values at most)
    wide = {n: k[".private_segment_fixed_size"] for n, k in ks.items() if re.search("ILi[0-9]+ELi[456]E", n)}
    assert len(wide) >= 48 and {n: b for n, b in wide.items() if b > 16} == {}
