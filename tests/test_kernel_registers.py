"""Registers of the sparse products, read from the metadata of the library built here: the
kernels of the hot loops stay within their launch bound without spilling to scratch."""

import os
import re
import struct
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
LIB = os.path.join(ROOT, "paper_2601_11338_amd", "libwalklap.so")
READELF = "/opt/rocm/llvm/bin/llvm-readelf"
MAGIC = b"__CLANG_OFFLOAD_BUNDLE__"


def code_objects(data):
    """The gfx950 code objects of the library's bundles."""
    at = data.find(MAGIC)
    while at >= 0:
        (count,) = struct.unpack_from("<Q", data, at + len(MAGIC))
        p = at + len(MAGIC) + 8
        for _ in range(count):
            off, size, n = struct.unpack_from("<QQQ", data, p)
            name = data[p + 24:p + 24 + n]
            p += 24 + n
            if b"gfx950" in name and size:
                yield data[at + off:at + off + size]
        at = data.find(MAGIC, at + 1)


def kernels(tmp_path):
    """{kernel name: (vector registers, spilled ones)}"""
    out = {}
    path = tmp_path / "code"
    for obj in code_objects(open(LIB, "rb").read()):
        path.write_bytes(obj)
        notes = subprocess.run([READELF, "--notes", str(path)], capture_output=True, text=True, check=True).stdout
        for k in notes.split("- .agpr_count:")[1:]:
            name = re.search(r"\.name:\s+(\S+)", k).group(1)
            out[name] = tuple(int(re.search(r"\.%s:\s+(\d+)" % f, k).group(1)) for f in ("vgpr_count", "vgpr_spill_count"))
    return out


def test_products_do_not_spill(tmp_path):
    if not (os.path.exists(LIB) and os.path.exists(READELF)):
        pytest.skip("library or llvm-readelf not there")
    found = kernels(tmp_path)
    # k_spmm<T, VW, LPN, G, MASK, E>: E = 1 (per-column coefficients with a running sum) is
    # faster with its four spilled registers than in any form without
    spmm = {n: s for n, (_, s) in found.items() if "k_spmmI" in n}
    assert len(spmm) > 100
    spilled = {n: s for n, s in spmm.items() if s > (4 if "ELi1EEEv" in n else 0)}
    assert not spilled
    # one and two FP64 columns: eight waves per SIMD
    narrow = {n: v for n, (v, _) in found.items() if re.search(r"k_spmmIdLi[12]ELi1ELi", n)}
    assert len(narrow) > 8 and max(narrow.values()) <= 64
