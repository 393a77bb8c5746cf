"""Registers of the built kernels, from the metadata of the library's own code
objects: forms whose speed rests on the compiler keeping them out of scratch or
within a number of waves per SIMD."""
import os
import struct

import pytest

LIB = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_1303_1377_amd", "libddamg.so")


def _code_objects(blob):
    """The gfx950 ELF files in the library's offload bundles."""
    magic = b"__CLANG_OFFLOAD_BUNDLE__"
    at = blob.find(magic)
    while at >= 0:
        pos = at + len(magic) + 8
        for _ in range(struct.unpack_from("<Q", blob, at + len(magic))[0]):
            off, size, n = struct.unpack_from("<QQQ", blob, pos)
            if b"gfx950" in blob[pos + 24 : pos + 24 + n] and size:
                yield blob[at + off : at + off + size]
            pos += 24 + n
        at = blob.find(magic, at + 1)


def _kernels():
    msgpack = pytest.importorskip("msgpack")
    if not os.path.exists(LIB):
        pytest.skip("library not built")
    out = {}
    for elf in _code_objects(open(LIB, "rb").read()):
        phoff, phentsize, phnum = struct.unpack_from("<Q", elf, 32)[0], *struct.unpack_from("<HH", elf, 54)
        for i in range(phnum):
            kind, _, off, _, _, size = struct.unpack_from("<IIQQQQ", elf, phoff + i * phentsize)
            end = off + size
            while kind == 4 and off < end:   # PT_NOTE
                nsz, dsz, typ = struct.unpack_from("<III", elf, off)
                data = off + 12 + (nsz + 3) // 4 * 4
                if typ == 32:   # AMDGPU metadata
                    for k in msgpack.unpackb(elf[data : data + dsz])["amdhsa.kernels"]:
                        out[k[".name"]] = k
                off = data + (dsz + 3) // 4 * 4
    assert out, "no kernel metadata in " + LIB
    return out


@pytest.fixture(scope="module")
def kernels():
    return _kernels()


def test_fine_sap_stays_in_registers(kernels):
    """Every form of the fine SAP, also of blocks with an extent of two beside longer
    ones, spills at most a few registers (the half sweep of such a block took up to
    1.36 times as long with 70 to 170 of them spilled)."""
    sap = {n: k for n, k in kernels.items() if "k_sap_fine" in n}
    assert len(sap) == 10
    for n, k in sap.items():
        assert k[".vgpr_spill_count"] <= 16 and k[".private_segment_fixed_size"] <= 128, n


def test_row_kernel_without_a_fold(kernels):
    """The row-split coarse stencil of FP16 storage keeps six waves per SIMD where it
    folds no Arnoldi step."""
    rows = [k for n, k in kernels.items() if "k_coarse_rowsIfDF16_" in n and "Lb1E" not in n]
    assert rows and all(k[".vgpr_count"] <= 80 for k in rows)
