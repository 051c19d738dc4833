"""Registers of the per-pixel decode kernel (k_dec_rows), read off the metadata
of the built library: an instance that takes a few registers too many loses a
wave per SIMD, which no result shows and which cost up to half of its speed."""
import re
import struct

import pytest

from paper_2602_12314_amd import build

msgpack = pytest.importorskip("msgpack")


def _kernels():
    """{mangled name: metadata} of every kernel: the code objects' AMDGPU notes
    (type 32, a msgpack map) hold them."""
    if build.needs_build():
        build.build()
    with open(build.LIB, "rb") as fh:
        blob = fh.read()
    out = {}
    for m in re.finditer(rb"AMDGPU\x00\x00", blob):
        namesz, descsz, kind = struct.unpack("<III", blob[m.start() - 12:m.start()])
        if (namesz, kind) != (7, 32):
            continue
        meta = msgpack.unpackb(blob[m.end():m.end() + descsz])
        out.update({k[".name"]: k for k in meta["amdhsa.kernels"]})
    return out


def _waves(meta):
    """Waves per SIMD that the registers allow: 512 of them (vector and
    accumulation registers together, which .vgpr_count is) in units of 8."""
    return min(8, 512 // (-(-meta[".vgpr_count"] // 8) * 8))


# least waves per SIMD of the 32-pixel block by (mode, E4M3), for D / 128 = 1 .. 8
INFER, LOSS, ADJ = 0, 1, 2
LEAST = {(INFER, 0): (7, 6, 4, 4, 2, 1, 2, 1), (INFER, 1): (4, 3, 2, 2, 2, 2, 2, 1),
         (LOSS, 0): (3, 3, 3, 3, 2, 1, 1, 1), (LOSS, 1): (2, 2, 2, 2, 2, 1, 1, 1),
         (ADJ, 0): (3, 3, 3, 3, 2, 1, 1, 1), (ADJ, 1): (2, 2, 2, 2, 2, 1, 2, 1)}


def test_rows_kernel_keeps_its_waves():
    seen = 0
    for name, meta in _kernels().items():
        m = re.search(r"k_dec_rowsINS_5TBF16ELi(\d)ELi(16|32)ELi(\d)ELb(\d)ELi(\d)ELi\dE", name)
        if not m:
            continue
        nt, d, mode, f8, nw = (int(x) for x in m.groups())
        least = LEAST[mode, f8][nt - 1] if nw == 4 else 2
        assert _waves(meta) >= least, (name, meta[".vgpr_count"], least)
        seen += 1
    assert seen == 2 * 3 * 2 * (8 + 4)  # d, mode, precision, D tiles of both block shapes
